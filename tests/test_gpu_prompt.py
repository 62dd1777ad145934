"""Prompt-time calls at the sizes where their work split can go wrong: the
request means (chunk windows, partial chunks, odd pages, unaligned values) and
the bulk append (tokens per workgroup, ragged remainders, skipped tokens) and
the writers of the 8-bit formats (rows per workgroup, rounding, alignment)."""

import numpy as np
import pytest
import torch

import paper_2609_33410_amd as F
from oracle import q8_oracle as q8
from workloads import host_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F.load_library()


def _pool(lens, hkv, page, d, seed):
    """Random pages and a block table in random page order."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    pages = [(n + page - 1) // page for n in lens]
    pool = torch.randn(sum(pages) + 1, hkv, page, d, generator=g, device="cuda").to(torch.bfloat16)
    perm = torch.randperm(sum(pages), generator=g, device="cuda").to(torch.int32)
    bt = torch.zeros(len(lens), max(max(pages), 1), dtype=torch.int32, device="cuda")
    first = 0
    for r, p in enumerate(pages):
        bt[r, :p] = perm[first:first + p]
        first += p
    return pool, bt


def _rows(pool, bt, r, n, page):
    """Logical rows [hkv, n, d] of sequence r in 64 bits."""
    t = pool[bt[r, :(n + page - 1) // page].long()].transpose(0, 1)
    return t.reshape(t.shape[0], -1, t.shape[3])[:, :n].double()


# lengths around the 16-key chunk, the wave stride (16 waves x 16 keys), the
# eight loads in flight and the 64-chunk block-table window of a wave (16384)
LENS = [0, 1, 15, 16, 17, 255, 256, 257, 2047, 2049, 16383, 16400, 17001]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("page", [16, 48, 64, 0])
@pytest.mark.parametrize("wide", [True, False])
def test_value_mean_lengths(d, page, wide):
    """FP32 sums of at most 2^15 values of a BF16 N(0,1): the error of a mean
    is below n 2^-24 max|v| / n < 1e-6 of the largest value (about 5)."""
    hkv = 3
    lens = LENS if page else [0, 1, 15, 17, 257, 2049, 17001]
    if page:
        v, bt = _pool(lens, hkv, page, d, d + page)
    else:
        v = torch.randn(len(lens), hkv, max(lens), d, device="cuda").to(torch.bfloat16)
        bt = None
    if not wide:  # the same rows two bytes past a 16-byte boundary
        shifted = torch.empty(v.numel() + 8, dtype=torch.bfloat16, device="cuda")
        off = 1 + (-shifted.data_ptr() // 2) % 8
        shifted[off:off + v.numel()] = v.view(-1)
        v = shifted[off:off + v.numel()].view(v.shape)
        assert v.data_ptr() % 16 == 2
    kv = F.kv_view(v, v, torch.tensor(lens, dtype=torch.int32, device="cuda"), num_kv_heads=hkv,
                   max_seq_len=max(lens), block_table=bt)
    got = F.fold_value_mean(kv, torch.full((len(lens), hkv, d), 7.0, device="cuda")).double()
    for r, n in enumerate(lens):
        x = _rows(v, bt, r, n, page) if page else v[r, :, :n].double()
        want = x.mean(1) if n else torch.zeros(hkv, d, dtype=torch.float64, device="cuda")
        assert (got[r] - want).abs().max().item() < 5e-6, (r, n)


def test_value_mean_skips_pages_outside_the_pool():
    v, bt = _pool([300, 40], 2, 16, 128, 3)
    bt[0, 3], bt[0, 7], bt[1, 0] = -1, v.shape[0], 10 ** 6
    kv = F.kv_view(v, v, torch.tensor([300, 40], dtype=torch.int32, device="cuda"),
                   num_kv_heads=2, max_seq_len=300, block_table=bt)
    got = F.fold_value_mean(kv, torch.empty(2, 2, 128, device="cuda")).double()
    for r, n in ((0, 300), (1, 40)):
        want = torch.zeros(2, 128, dtype=torch.float64, device="cuda")
        for p in range((n + 15) // 16):
            page = int(bt[r, p])
            if 0 <= page < v.shape[0]:
                want += v[page, :, :min(16, n - 16 * p)].double().sum(1)
        assert (got[r] - want / n).abs().max().item() < 5e-6


@pytest.mark.parametrize("d,seqs", [(128, (1 << 14) + 1), (64, (1 << 15) + 1)])
def test_value_mean_of_more_pairs_than_one_launch_holds(d, seqs):
    """64 heads of just over 2^14 (D = 64: 2^15) sequences: four (two)
    workgroups of 1024 threads a pair would pass the 2^32 threads of a launch.
    Rows of at most 16 keys, on one of four pages."""
    hkv, page = 64, 16
    g = torch.Generator(device="cuda").manual_seed(d)
    v = torch.randn(4, hkv, page, d, generator=g, device="cuda").to(torch.bfloat16)
    bt = torch.randint(0, 4, (seqs, 1), generator=g, device="cuda").to(torch.int32)
    lens = torch.randint(0, page + 1, (seqs,), generator=g, device="cuda").to(torch.int32)
    kv = F.kv_view(v, v, lens, num_kv_heads=hkv, max_seq_len=page, block_table=bt)
    got = F.fold_value_mean(kv, torch.full((seqs, hkv, d), 7.0, device="cuda"))
    sums = torch.cat([torch.zeros_like(v[:, :, :1]).double(), v.double().cumsum(2)], 2)
    want = (sums / torch.arange(page + 1, device="cuda").clamp(min=1)[:, None]).float()
    want = want.transpose(1, 2).contiguous()  # [page, length, hkv, d]
    for i in range(0, seqs, 1 << 12):
        part = slice(i, min(i + (1 << 12), seqs))
        err = got[part] - want[bt[part, 0].long(), lens[part].long()]
        assert err.abs().max().item() < 5e-6, i


@pytest.mark.parametrize("d,hkv,n_tok", [(128, 3, 1), (128, 8, 2048), (128, 8, 2049), (64, 5, 6554),
                                         (64, 1, 32769), (128, 7, 2341)])
@pytest.mark.parametrize("which", ["kv", "k", "v"])
def test_append_whole_prompts(d, hkv, n_tok, which):
    """Counts on both sides of the four-rows-per-thread line (16384 rows at D =
    128, 32768 at D = 64) and remainders of a workgroup; skipped tokens in
    between leave every other row alone."""
    page = 16
    lens = [n_tok // 3, n_tok - n_tok // 3]
    pool, bt = _pool([max(1, n) for n in lens], hkv, page, d, n_tok)
    bad = bt.shape[1] - 1
    if n_tok > 100:
        bt[1, bad] = -5
    k, v = torch.full_like(pool, 3.0), torch.full_like(pool, 3.0)
    src = torch.randn(2, n_tok, hkv, d, device="cuda").to(torch.bfloat16)
    seq = torch.cat([torch.full((n,), i) for i, n in enumerate(lens)]).to(torch.int32)
    pos = torch.cat([torch.arange(n) for n in lens]).to(torch.int32)
    if n_tok > 100:
        seq[50], seq[51], pos[52], pos[53] = -1, 2, -3, bt.shape[1] * page
    kv = F.kv_view(k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"), num_kv_heads=hkv,
                   max_seq_len=max(lens), block_table=bt)
    F.fold_append_kv(kv, src[0] if "k" in which else None, src[1] if "v" in which else None,
                     seq.cuda(), pos.cuda(), k if "k" in which else None,
                     v if "v" in which else None)
    seq, pos, table = seq.long(), pos.long(), bt.cpu().long()
    cap = min(table.shape[1] * page, max(lens))
    ok = (seq >= 0) & (seq < 2) & (pos >= 0) & (pos < cap)
    phys = torch.full_like(seq, -1)
    phys[ok] = table[seq[ok], pos[ok] // page]
    ok &= phys >= 0
    for cache, rows, on in ((k, src[0], "k" in which), (v, src[1], "v" in which)):
        want = torch.full_like(pool, 3.0)
        if on:
            at = ok.nonzero()[:, 0].cuda()
            want[phys[ok].cuda(), :, (pos[ok] % page).cuda()] = rows[at]
        assert torch.equal(cache, want)


def _shifted(t, wide):
    """t itself, or a copy of it two bytes past a 16-byte boundary."""
    if wide:
        return t
    raw = torch.empty(t.numel() * t.element_size() + 32, dtype=torch.uint8, device="cuda")
    off = (-raw.data_ptr()) % 16 + 2
    out = raw[off:off + t.numel() * t.element_size()].view(t.dtype).view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 2
    return out


def _write_all(fn, src, arrays, hkv, wide):
    """Token i of src [n, hkv, d] written to position i of one contiguous
    sequence of planes [1, hkv, n, d]; returns the planes."""
    n, _, d = src.shape
    planes = [_shifted(torch.full((1, hkv, n, d) if full else (1, hkv, n), 0x33, dtype=dt,
                                  device="cuda"), wide) for dt, full in arrays]
    kv = F.kv_view(planes[0].view(torch.int8), None,
                   torch.tensor([n], dtype=torch.int32, device="cuda"), num_kv_heads=hkv,
                   max_seq_len=n, k_is_layout_only=True)
    fn(kv, _shifted(src, wide), torch.zeros(n, dtype=torch.int32, device="cuda"),
       torch.arange(n, dtype=torch.int32, device="cuda"), planes)
    return [p[0].transpose(0, 1).cpu().numpy() for p in planes]


def _write_keys(kv, src, seq, pos, planes):
    F.fold_q8_write_keys(kv, src, seq, pos, F.Q8Keys(*planes))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hkv,n", [(1, 1), (3, 11), (1, 32), (1, 65), (5, 333), (7, 301)])
@pytest.mark.parametrize("wide", [True, False])
def test_key_writer_rounding(d, hkv, n, wide):
    """Codes of keys whose quotients tie (one-hot rows, small integers), span
    many binades or are tiny, zero or large: the oracle's, bit for bit."""
    g = torch.Generator().manual_seed(n + d)
    k = torch.randn(n, hkv, d, generator=g)
    pick = torch.arange(n * hkv).view(n, hkv, 1) % 8
    one_hot = torch.zeros(n, hkv, d).scatter_(
        2, torch.randint(0, d, (n, hkv, 1), generator=g), 127.0)
    few = torch.randint(-3, 4, (n, hkv, d), generator=g).float()
    wide_span = k * torch.exp2(torch.randint(-14, 15, (n, hkv, d), generator=g).float())
    for i, other in enumerate((one_hot, few, wide_span, torch.zeros_like(k), k * 2.0 ** -120,
                               k * 2.0 ** 100)):
        k = torch.where(pick == i + 1, other, k)
    k = k.to(torch.bfloat16)
    got = _write_all(_write_keys, k.cuda(), [(torch.int8, True), (torch.int8, True),
                                             (torch.int16, False)], hkv, wide)
    a, b, e = q8.split_keys(host_bits(k))
    assert np.array_equal(got[0], a) and np.array_equal(got[1], b)
    assert np.array_equal(got[2].view(np.uint16), e)


def test_key_writer_keeps_non_finite_keys_to_themselves():
    """A key with an infinity or a NaN changes no other key's code; a NaN key
    is stored as zero."""
    k = torch.randn(40, 2, 128).to(torch.bfloat16)
    clean = _write_all(_write_keys, k.cuda(), [(torch.int8, True), (torch.int8, True),
                                               (torch.int16, False)], 2, True)
    k[7, 0, 5], k[21, 1, 100], k[22, 0, 0] = float("inf"), float("nan"), float("-inf")
    got = _write_all(_write_keys, k.cuda(), [(torch.int8, True), (torch.int8, True),
                                             (torch.int16, False)], 2, True)
    ok = np.ones((40, 2), dtype=bool)
    ok[7, 0] = ok[21, 1] = ok[22, 0] = False
    for x, y in zip(got, clean):
        assert np.array_equal(x[ok], y[ok])
    assert not got[0][21, 1].any() and not got[1][21, 1].any() and got[2][21, 1] == 0


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("wide", [True, False])
def test_key_writer_forms_agree_on_extreme_keys(d, wide):
    """More than 2048 rows take the row groups, fewer a wave a row: the same
    codes and scales for infinities, NaN, the largest and the smallest values,
    and the oracle's for every finite key beside them."""
    inf, nan, most = float("inf"), float("nan"), 3.3895313892515355e38
    k = torch.randn(1100, 2, d, generator=torch.Generator().manual_seed(d))
    k[3, 0, 5], k[4, 1, d - 1] = inf, -inf
    k[5, 0, 0], k[5, 0, 1] = inf, inf
    k[6, 1, 2], k[6, 1, d - 3] = inf, -inf
    k[7, 0, 9], k[8, 1, 0], k[8, 1, 4] = nan, nan, inf
    k[9] = most
    k[10, :, ::2], k[10, :, 1::2] = most, -most
    k[11], k[12] = 2.0 ** -133, 2.0 ** -126
    k[1099, 1] = inf
    k = k.to(torch.bfloat16)
    arrays = [(torch.int8, True), (torch.int8, True), (torch.int16, False)]
    got = _write_all(_write_keys, k.cuda(), arrays, 2, wide)
    few = _write_all(_write_keys, k[:40].contiguous().cuda(), arrays, 2, wide)
    for x, y in zip(got, few):
        assert np.array_equal(x[:40], y)
    ok = torch.isfinite(k.float()).all(-1).numpy()
    ok[9:11] = False  # the codes' scale passes the largest BF16
    want = q8.split_keys(host_bits(torch.where(torch.from_numpy(ok)[..., None], k, 0)))
    for x, y in zip(got, want):
        assert np.array_equal(x.view(y.dtype)[ok], y[ok])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale_exp", [-6, 0, 3])
@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("copies", [1, 9])
def test_value_writer_every_bf16(d, scale_exp, wide, copies):
    """The E4M3 planes of every BF16 pattern (NaN codes only checked to be the
    saturated ones), of 3 heads' rows: once, the form of up to 2^19 elements,
    and nine times, a prompt's, with a ragged last workgroup."""
    bits = torch.arange(65536, dtype=torch.int32).to(torch.int16)
    pad = (-65536 * copies) % (3 * d) + (3 * d if copies > 1 else 0)
    v = torch.cat([bits.repeat(copies), bits[:pad]]).view(torch.bfloat16).view(-1, 3, d)
    assert (v.numel() > 2 ** 19) == (copies > 1)
    got = _write_all(lambda kv, s, seq, pos, pl: F.fold_v8_write_values(
        kv, s, seq, pos, F.V8Values(pl[0], pl[1], scale_exp)), v.cuda(),
        [(torch.uint8, True), (torch.uint8, True)], 3, wide)
    nan = torch.isnan(v.float()).numpy()
    with np.errstate(all="ignore"):
        p, r = q8.split_values(np.where(nan, 0, host_bits(v)).astype(np.uint16), scale_exp)
    assert np.array_equal(got[0][~nan], p[~nan]) and np.array_equal(got[1][~nan], r[~nan])
    assert ((got[0][nan] & 0x7F) == 0x7E).all()
