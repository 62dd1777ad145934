"""The combine at the slot counts where its batches of loads change."""

import pytest
import torch

import paper_2609_33410_amd as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("slots", [1, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 65, 97])
@pytest.mark.parametrize("model,shift,out_dtype",
                         [(False, 0, torch.float32), (True, 0, torch.float32),
                          (True, 1, torch.float32), (False, 0, torch.bfloat16),
                          (False, 1, torch.bfloat16)])
def test_slots_add_in_order(slots, d, model, shift, out_dtype):
    """A, L and the cut mass are FP32 sums in increasing slot order: L's
    log-sum-exp and the sum of A are the sequential sums, the output their
    quotient to an FP32 division (and, with the model, one fused add that the
    reference rounds twice: 2^-22 of the terms' magnitudes; BF16 outputs add
    half a unit in the last of 8 significant bits: 2^(e-8) <= 2^-8 |x| for x
    in [2^e, 2^(e+1))).  Nine rows leave the last wave part empty; shift moves
    the arrays off the 16-byte lines."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    heads, hkv, rows = 3, 1, 9

    def dev(t):
        flat = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
        return flat[shift:].view(t.shape).copy_(t)

    gen = torch.Generator().manual_seed(slots + d)
    A = torch.randn(slots, rows, d, generator=gen) * 3
    L = torch.rand(slots, rows, generator=gen) + 0.25
    cut = torch.rand(slots, rows, generator=gen)
    mean = torch.randn(rows // heads, hkv, d, generator=gen)
    z = torch.randn(rows, generator=gen)
    acc, l, c = torch.zeros(rows, d), torch.zeros(rows), torch.zeros(rows)
    for s in range(slots):
        acc, l, c = acc + A[s], l + L[s], c + cut[s]
    mag = acc.abs()
    if model:
        m = mean.repeat_interleave(heads // hkv, 1).reshape(rows, d)
        mag = mag + (c[:, None] * m).abs()
        acc = acc + c[:, None] * m
    out = dev(torch.empty(rows // heads, heads, d, dtype=out_dtype))
    lse = torch.empty(rows, device="cuda")
    cert = torch.empty(rows, dtype=torch.uint8, device="cuda")
    extra = dict(part_Lcut=cut.view(slots, -1, heads).cuda(), mean=dev(mean)) if model else {}
    F.fold_combine(dev(A.view(slots, -1, heads, d)), L.view(slots, -1, heads).cuda(), out,
                   z=z.cuda(), lse_out=lse, cert_out=cert, **extra)
    torch.cuda.synchronize()
    tol = 2.0 ** -22 * (mag / l[:, None])
    if out_dtype == torch.bfloat16:
        tol = tol + 2.0 ** -8 * (acc / l[:, None]).abs()
    assert ((out.cpu().float().view(rows, d) - acc / l[:, None]).abs() <= tol).all()
    assert (lse.cpu() - (z + torch.log2(l))).abs().max() <= 2e-6 * (1 + l.log2().abs().max())
    assert torch.equal(cert.cpu(), (l < 0.5).to(torch.uint8))
