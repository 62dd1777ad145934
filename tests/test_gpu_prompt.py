"""Prompt-time calls at the sizes where their work split can go wrong: the
request means (chunk windows, partial chunks, odd pages, unaligned values) and
the bulk append (tokens per workgroup, ragged remainders, skipped tokens)."""

import pytest
import torch

import paper_2609_33410_amd as F

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
