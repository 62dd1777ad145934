"""Scans that take the longest sequences first (with more than one row, those of
one split below): every sequence is scanned by its own workgroups,
whatever the lengths and their count."""

import pytest
import torch

import paper_2609_33410_amd as F

pytestmark = pytest.mark.gpu

PAGE, PAGES = 16, 33  # 528 keys: eight chunks a wave in one split; leading bits 512 + 16


def _lens(kind, n):
    g = torch.Generator().manual_seed(n)
    cap = PAGE * PAGES
    if kind == "equal":
        return torch.full((n,), 300)
    if kind == "random":
        return torch.randint(0, cap + 1, (n,), generator=g)
    if kind == "near":  # apart in the bits the order looks at, and below them
        base = torch.tensor([0, 1, 2, 3, 4, 15, 16, 17, 63, 64, 65, 127, 128, 255, 256, 257, 511, 512, cap])
        return base[torch.randint(0, len(base), (n,), generator=g)]
    out = torch.randint(0, cap + 1, (n,), generator=g)  # past the capacity, below zero
    out[torch.randint(0, n, (n // 2,), generator=g)] = cap + 1000
    out[0], out[n - 1] = -5, 2 ** 31 - 1
    return out


@pytest.mark.parametrize("kind", ["equal", "random", "near", "clamped"])
@pytest.mark.parametrize("n", [2, 3, 17, 33, 63, 64])
@pytest.mark.parametrize("scan,hkv,group,splits", [("bf16", 3, 1, 2), ("two-plane", 3, 1, 3),
                                                   ("two-plane", 3, 4, 2), ("two-plane", 1, 16, 3),
                                                   ("two-plane", 2, 2, 5), ("two-plane", 3, 4, 1),
                                                   ("two-plane", 1, 16, 1)])
def test_every_sequence_is_scanned_once(kind, n, scan, hkv, group, splits):
    """The slots of a batch are, bit for bit, those of its sequences alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d, h = 64, hkv * group
    g = torch.Generator(device="cuda").manual_seed(n)
    k = torch.randn(40, hkv, PAGE, d, generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn(40, hkv, PAGE, d, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(n, h, d, generator=g, device="cuda").to(torch.bfloat16)
    bt = torch.randint(0, 40, (n, PAGES), generator=g, device="cuda").to(torch.int32)
    lens = _lens(kind, n).to(torch.int32).cuda()
    z = torch.full((n, h), 2.0, device="cuda")
    a = torch.randint(-127, 128, (2, 40, hkv, PAGE, d), generator=g, device="cuda").to(torch.int8)
    keys = F.Q8Keys(a[0], a[1], torch.full((40, hkv, PAGE), 0x3D00, dtype=torch.int16,
                                           device="cuda"))

    def slots(at):
        part_a = torch.full((splits, at.stop - at.start, h, d), float("nan"), device="cuda")
        part_l = torch.full((splits, at.stop - at.start, h), float("nan"), device="cuda")
        args = dict(num_kv_heads=hkv, max_seq_len=PAGE * PAGES, block_table=bt[at])
        if scan == "bf16":
            kv = F.kv_view(k, v, lens[at], **args)
            F.fold_decode_split(kv, F.q_view(q[at]), 0.125, z[at], 16.0, splits, 0, part_a, part_l)
        else:
            kv = F.kv_view(a[0], v, lens[at], k_is_layout_only=True, **args)
            qq = F.q8_empty_query(q[at])
            F.fold_q8_split_query(q[at], 0.125, qq, req_lens=lens[at], kappa=-4.0)
            F.fold_q8_decode_split(kv, keys, qq, z[at], 16.0, splits, 0, part_a, part_l)
        return part_a, part_l

    all_a, all_l = slots(slice(0, n))
    for i in range(n):
        one_a, one_l = slots(slice(i, i + 1))
        assert torch.equal(all_a[:, i], one_a[:, 0]) and torch.equal(all_l[:, i], one_l[:, 0]), i
