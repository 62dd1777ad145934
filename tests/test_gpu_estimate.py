"""The estimate's sample positions with and without a power of two in its two
rules (strata, page size), for stratified and short rows, and its sort over a
full and a partly filled network."""

import numpy as np
import pytest
import torch

import paper_2609_33410_amd as F
from oracle import estimate_level
from tests import _adapt, _gpu
from workloads import make_custom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F.load_library()


@pytest.mark.parametrize("strata", [1, 64, 96, 127, 128, 256])
@pytest.mark.parametrize("page,group,d", [(16, 16, 64), (48, 4, 128), (64, 1, 64), (0, 8, 128)])
def test_samples_match_the_oracle(strata, page, group, d):
    """Rows one key short of, at and past the stratified rule, and long odd
    ones.  Scores of a few tens of binades accumulate in FP32 over D products:
    Z agrees to 1e-3 binades (as the other estimate tests ask), while one
    sample taken a key off moves a centre score by binades."""
    params = {"sink": 16, "recent": 48, "strata": strata, "trim_lo": min(2, strata - 1),
              "trim_hi": min(5, max(0, strata - 3))}
    full = 64 + strata
    lens = [full - 1, full, full + 1, full + 17, 0, 1003, 6007]
    wl = make_custom(batch=len(lens), heads=2 * group, kv_heads=2, dim=d, lens=lens,
                     paged=page > 0, page_size=page or 16, spike_count=20, n_sink=2,
                     seed=strata + group, device="cuda")
    _, flat = _gpu.kv_views(wl, with_v=False)
    z = torch.empty(wl.batch, wl.num_heads, dtype=torch.float32, device="cuda")
    F.fold_ref_estimate(flat, F.q_view(wl.q), wl.sm_scale, z, params=params)
    torch.cuda.synchronize()
    oi = _adapt.oracle_inputs(wl)
    zo = estimate_level(oi["q_bits"], oi["k_bits"], num_kv_heads=oi["num_kv_heads"],
                        page_size=oi["page_size"], sm_scale=oi["sm_scale"],
                        seq_lens=oi["flat"]["seq_lens"], block_table=oi["flat"]["block_table"],
                        p=params)
    assert np.abs(z.cpu().double().numpy() - zo).max() <= 1e-3


def test_front_of_more_groups_than_sixteen_waves_allow():
    """2^22 groups of 16 rows: workgroups of 1024 threads would reach 2^32
    threads, past a launch's limit.  64 requests' queries repeated: every
    repetition has the codes, eta, tau and Z of the 64 alone."""
    reqs, heads, hkv, d, rep = 64, 1024, 64, 64, 1 << 10
    g = torch.Generator(device="cuda").manual_seed(22)
    k = torch.randn(64 * 64, hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(reqs, heads, d, generator=g, device="cuda").to(torch.bfloat16)
    lens = torch.randint(0, 65, (reqs,), generator=g, device="cuda").to(torch.int32)
    bt = torch.randint(0, 256, (reqs, 4), generator=g, device="cuda").to(torch.int32)
    plane = torch.empty(256, hkv, 16, d, dtype=torch.int8, device="cuda")
    keys = F.Q8Keys(plane, torch.empty_like(plane),
                    torch.empty(256, hkv, 16, dtype=torch.int16, device="cuda"))
    pool = F.kv_view(plane, None, torch.full((256,), 16, dtype=torch.int32, device="cuda"),
                     num_kv_heads=hkv, max_seq_len=16, k_is_layout_only=True)
    at = torch.arange(4096, device="cuda", dtype=torch.int32)
    F.fold_q8_write_keys(pool, k, at // 16, at % 16, keys)

    def front(n):
        qn = q.repeat(n, 1, 1)
        kv = F.kv_view(plane, None, lens.repeat(n), num_kv_heads=hkv, max_seq_len=64,
                       block_table=bt.repeat(n, 1), k_is_layout_only=True)
        qq = F.q8_empty_query(qn)
        z = torch.full((n * reqs, heads), float("nan"), device="cuda")
        F.fold_q8_front(kv, keys, qn, 0.125, qq, z, req_lens=kv.tensors[2])
        return qq.planes, qq.eta, qq.tau, z

    want = front(1)
    assert torch.isfinite(want[3]).all()
    for got, w in zip(front(rep), want):
        got = got.view(rep, *w.shape)
        for i in range(0, rep, 64):
            assert torch.equal(got[i:i + 64], w.expand(64, *w.shape)), i
