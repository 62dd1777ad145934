"""The two-plane scan of 2 to 16 rows at the sizes where its stream, list and
in-place refinement can go wrong: block-table windows of 64 chunks a wave, odd
steps, odd pages and unaligned contiguous rows, packed and unpacked row counts,
steps that list a few keys and steps that refine them all."""

import numpy as np
import pytest
import torch

import paper_2609_33410_amd as F
from oracle import q8_oracle as q8
from tests import _adapt, _gpu_q8
from tests.test_gpu_q8 import INF, _full_parity
from tests.test_gpu_v8 import _v8_parity
from workloads import host_bits, make_cascade, make_custom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F.load_library()


@pytest.mark.parametrize("d,group,page", [(64, 2, 48), (128, 4, 16), (128, 16, 32), (64, 16, 16)])
def test_windows_and_odd_steps(d, group, page):
    """One split of 4096 + 16 k keys: a wave's second window starts with its
    65th chunk; chunk counts leave whole, odd and partial last steps."""
    lens = [4095, 4097, 4160, 4096 + 16 * 5 + 3, 31]
    wl = make_custom(batch=len(lens), heads=group, kv_heads=1, dim=d, lens=lens, page_size=page,
                     spike_count=30, n_sink=1, seed=d + group, device="cuda")
    for T, kappa in ((INF, -4.0), (16.0, -4.0), (8.0, 3.0)):
        _full_parity(wl, T, kappa=kappa, splits=[1], own_mode=False)


@pytest.mark.parametrize("group", [2, 8, 16])
@pytest.mark.parametrize("kappa", [-8.0, 0.0, 2.0, INF])
def test_listed_and_refined_in_place(group, kappa):
    """Refine thresholds from a key here and there to every key: list entries
    that wrap, gathers inside the stream, steps refined in place; 8-bit values
    with their second plane through both."""
    lens = [700, 1337]
    wl = make_custom(batch=2, heads=2 * group, kv_heads=2, dim=128, lens=lens, spike_count=40,
                     n_sink=2, seed=int(group + 10 * min(kappa, 9.0)) % 97, device="cuda")
    for T in (INF, 16.0, 5.0):
        _full_parity(wl, T, kappa=kappa, splits=[2], own_mode=False)
        _v8_parity(wl, T, kappa_v=kappa, splits=[2])


@pytest.mark.parametrize("group,d", [(2, 128), (8, 64), (8, 128), (16, 128), (16, 64)])
@pytest.mark.parametrize("kappa", [-6.0, 1.0])
def test_waves_of_one_step_and_two(group, d, kappa):
    """Waves of no chunk, one step (refined in place) and two: the prologue's
    two steps are all of the scan, and the gather runs once, after the last."""
    lens = [256, 300, 97, 1, 520]
    wl = make_custom(batch=len(lens), heads=2 * group, kv_heads=2, dim=d, lens=lens, spike_count=20,
                     n_sink=1, seed=group + d, device="cuda")
    for T in (INF, 10.0):
        for splits in ([2], [5]):  # five: at most one step a wave, by the view's capacity
            _full_parity(wl, T, kappa=kappa, splits=splits, own_mode=False)
            _v8_parity(wl, T, kappa_v=kappa, splits=splits)


@pytest.mark.parametrize("requests,heads,kv_heads", [(2, 8, 2), (3, 8, 2), (3, 4, 1), (4, 8, 2),
                                                     (5, 2, 1)])
def test_stacked_rows_around_eight(requests, heads, kv_heads):
    """Levels of 8, 12 and 16 stacked rows (and 10): several requests' GQA
    groups in one row block, packed two chunks a pass up to eight rows."""
    wl = make_cascade(requests=requests, heads=heads, kv_heads=kv_heads, dim=64, prefix_len=816,
                      suffix_len=32, splits=(2, 1), seed=requests + heads, device="cuda")
    for T in (INF, 10.0):
        _full_parity(wl, T, kappa=1.0, own_mode=False)


@pytest.mark.parametrize("T", [INF, 16.0])
def test_a_page_outside_the_pool_touches_its_sequence_only(T):
    wl = make_custom(batch=3, heads=8, kv_heads=2, dim=128, lens=[400, 333, 200], spike_count=5,
                     n_sink=1, seed=8, device="cuda")
    res, keys = _gpu_q8.run(wl, T, kappa=-4.0, splits=[2])
    for lv in wl.levels:
        lv.block_table[1, 3], lv.block_table[1, 9] = -1, 10 ** 6
    bad, _ = _gpu_q8.run(wl, T, kappa=-4.0, splits=[2], keys=keys, z=res["z"].cuda())
    for r in (0, 2):
        assert torch.equal(bad["out"][r], res["out"][r])
    assert torch.isfinite(bad["out"][1]).all()


@pytest.mark.parametrize("group,d", [(2, 128), (8, 64), (8, 128), (16, 128), (16, 64)])
@pytest.mark.parametrize("kappa", [-4.0, INF])
@pytest.mark.parametrize("T", [INF, 16.0])
def test_an_infinite_value_stays_infinite(group, d, kappa, T):
    """A refined key (listed at kappa = -4, refined in place at inf) and, at
    full depth, one that is not, each with an infinite value in a channel of its
    own: those channels of the rows that weigh the key are infinite, as 0 times
    infinity must enter no sum, and every other output keeps its bits."""
    wl = make_custom(batch=2, heads=2 * group, kv_heads=2, dim=d, lens=[700, 333],
                     spike_count=6, n_sink=1, seed=group + d, device="cuda")
    ref, keys = _gpu_q8.run(wl, T, kappa=kappa, splits=[2], debug=True)
    clean, _ = _gpu_q8.run(wl, T, kappa=kappa, splits=[2], keys=keys)
    bits = ref["dbg"][0]["refine_gate_out"][0, 1, 0, :700]
    refined = int((bits == 1).nonzero()[0])
    plain = int((bits == 0).nonzero()[0]) if kappa < INF and T == INF else None
    x = ref["dbg"][0]["x_out"][0, group:]  # request 0, kv head 1
    assert bool((x[:, refined] > -60).all()) or T < INF
    hit = {5: refined, 9: plain}
    for ch, key in hit.items():
        if key is not None:
            page = int(wl.levels[0].block_table[0, key // wl.page_size])
            wl.v[page, 1, key % wl.page_size, ch] = float("inf") if ch == 5 else float("-inf")
    got, _ = _gpu_q8.run(wl, T, kappa=kappa, splits=[2], keys=keys)
    out, want = got["out"], clean["out"].clone()
    if T == INF:
        want[0, group:, 5] = float("inf")
        if plain is not None:
            want[0, group:, 9] = float("-inf")
        assert torch.equal(out, want)
    else:  # a row that cuts the key shares the group's read: its channel is left out
        live = x[:, refined] >= -T
        assert live.any() and bool((out[0, group:, 5][live] == float("inf")).all())
        want[0, group:, 5] = out[0, group:, 5] = 0.0
        assert torch.equal(out, want)


@pytest.mark.parametrize("group", [4, 16])
@pytest.mark.parametrize("kappa", [-4.0, INF])
def test_scores_of_a_tiny_query_scale(group, kappa):
    """Queries of 2^-112 on keys of 2^112: eta is near 2^-123, the smallest
    scale FP32 holds in full, and keeps all its bits (L to 2e-5)."""
    wl = make_custom(batch=2, heads=2 * group, kv_heads=2, dim=128, lens=[500, 333],
                     spike_count=6, n_sink=1, seed=group, device="cuda")
    wl.q = (wl.q.float() * 2.0 ** -112).to(torch.bfloat16)
    wl.k = (wl.k.float() * 2.0 ** 112).to(torch.bfloat16)
    oi = _adapt.oracle_inputs(wl)
    res, keys = _gpu_q8.run(wl, INF, kappa=kappa, splits=[2])
    eta = res["eta"]
    assert eta.min() >= 2.0 ** -126 and eta.max() < 2.0 ** -118
    planes = q8.split_keys(host_bits(wl.k))
    qa, qb, eta = q8.split_queries(host_bits(wl.q), wl.sm_scale)
    tau = np.array([q8.refine_tau(n, kappa) for n in wl.flat.seq_lens_host], dtype=np.float32)
    _, pl = q8.decode_level_q8(qa, qb, eta, planes, oi["v_bits"], num_kv_heads=2,
                               page_size=wl.page_size, z=res["z"].double().numpy(), T=INF, tau=tau,
                               num_splits=2, **oi["levels"][0])
    got = res["part_L"].double().numpy()
    print("  L error", np.abs(got / pl - 1).max())
    assert np.allclose(got, pl, rtol=2e-5, atol=0)


@pytest.mark.parametrize("group", [2, 8, 16])
@pytest.mark.parametrize("values8", [False, True])
@pytest.mark.parametrize("kappa", [-4.0, 0.0, INF])
@pytest.mark.parametrize("splits", [2, 11])
def test_cut_masses_of_the_production_scan(splits, group, values8, kappa):
    """Cut masses asked for without debug outputs, of keys that stay in the
    stream, are listed or refined in place: the debug variant's slots bit for
    bit, and the sum of the cut weights of its exported scores (FP32 sums of
    at most 1337 terms: 2e-5).  Eleven splits leave a wave at most one step, which
    the production scan serves with a kernel of its own."""
    wl = make_custom(batch=2, heads=2 * group, kv_heads=2, dim=128, lens=[700, 1337],
                     spike_count=40, n_sink=2, seed=group, device="cuda")
    keys = _gpu_q8.encode_cache(wl)
    vals = _gpu_q8.encode_values(wl) if values8 else None
    qq = _gpu_q8.split_query(wl, kappa, kappa)
    levels, _ = _gpu_q8.level_views(wl, keys)
    z = _gpu_q8.estimate(wl, keys, qq)
    b, h, d = wl.q.shape

    def scan(T, **debug):
        out = [torch.full(s, float("nan"), device="cuda") for s in ((splits, b, h, d), (splits, b, h), (splits, b, h))]
        F.fold_q8_decode_split(levels[0], keys, qq, z, T, splits, 0, out[0], out[1], part_Lcut=out[2],
                               values=vals, **debug)
        return out

    for T in (INF, 8.0):
        x = torch.full((b, h, 1337), -INF, device="cuda")
        want = scan(T, x_out=x)
        got = scan(T)
        for g, w in zip(got, want):
            assert torch.equal(g, w)
        x = x.double()
        cut = torch.where(x < -T, torch.exp2(x), torch.zeros_like(x)).sum(-1)
        assert T == INF or bool((cut > 0).all())
        assert torch.allclose(got[2].double().sum(0), cut, rtol=2e-5, atol=0)
