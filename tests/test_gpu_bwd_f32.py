"""GPU parity of the fp32 attention backward, whose waves take every fourth tile of a 32-row block, or all of them
where many blocks of few tiles fill the chip: fewer tiles than waves, one more than a multiple, ragged last tiles,
groups of query heads.  The bars are those of the backward tests (1e-4 relative L2 per matrix
against the fp64 oracle)."""
import pytest
import torch

from paper_2609_34866_amd import jab

from test_gpu_backward import _check_backward
from test_gpu_kl_bwd import _check_kl_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [16, 64, 128])
@pytest.mark.parametrize("B,T,hq,hkv", [(1, 20, 2, 2), (2, 33, 4, 2), (1, 161, 2, 2), (1, 130, 4, 1), (8, 64, 2, 1),
                                        (150, 40, 4, 4), (130, 70, 8, 2)])
def test_fp32_backward_matches_oracle(B, T, hq, hkv, dh):
    shape = (B, T, 64, hq, hkv, dh, 32, "f32")
    _check_backward(shape)
    _check_kl_backward(shape + (0.0, 0.1))


def test_more_workgroups_than_one_launch_takes():
    """64 heads of 262144 one-token sequences: 2^24 workgroups of 256 threads, one more than a grid dimension
    holds.  With one token P = 1, so dV is the output gradient summed over the group and dS = 0 up to the
    rounding of the two sums whose difference it is."""
    B, d, hq, hkv, dh = 262144, 32, 64, 16, 16
    p = jab.problem(B, 1, d, hq, hkv, dh, 32, torch.float32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.randn((B, 1, d), generator=gen, device="cuda")
    w = torch.randn((p.rows, d), generator=gen, device="cuda") * 0.1
    bits = (3, 3, 3)
    scale, zero = jab.quant_init(p, w, bits)
    a, qk, lse = jab.attn_ref_kl(p, x, w)
    gam = jab.lsq_gscale(bits, 32)
    w_hat = jab.quantize(p, w, bits, scale, zero)["w_hat"]
    xs = x.reshape(B, d).double()
    diff = xs @ (w_hat - w)[-hkv * dh:].double().t().contiguous()        # [B][hkv dh], the same for a group's heads
    want = (diff.t().contiguous() @ xs) * ((hq // hkv) * 2.0 / (B * hq * dh))
    for dw in (jab.loss_bwd(p, x, w, bits, scale, zero, a, gam)[1],
               jab.loss_bwd_kl(p, x, w, bits, scale, zero, a, qk, lse, gam, 0.1)[1]):
        dv = dw[-hkv * dh:].double()
        # 2^-24 per addition, 262144 of them in up to sixteen parts
        assert float((dv - want).norm()) <= 1e-4 * float(want.norm())
        assert float(dw[:-hkv * dh].double().norm()) <= 1e-4 * float(want.norm())


@pytest.mark.parametrize("dh", [16, 64, 128])
@pytest.mark.parametrize("B,T,hq,hkv", [(1, 161, 4, 2), (8, 512, 12, 12), (20, 100, 12, 12), (150, 40, 4, 4), (16, 100, 8, 2)])
def test_lambda_zero_is_the_plain_backward(B, T, hq, hkv, dh):
    """The KL form takes the same number of waves and the same order of sums: equal bits, for blocks of one wave
    and of four."""
    p = jab.problem(B, T, 64, hq, hkv, dh, 32, torch.float32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x = torch.randn((B, T, 64), generator=gen, device="cuda")
    w = torch.randn((p.rows, 64), generator=gen, device="cuda") * 0.1
    bits = (3, 4, 2)
    scale, zero = jab.quant_init(p, w, bits)
    a, qk, lse = jab.attn_ref_kl(p, x, w)
    gam = jab.lsq_gscale(bits, 32)
    _, dw, ds = jab.loss_bwd(p, x, w, bits, scale, zero, a, gam)
    _, dw0, ds0 = jab.loss_bwd_kl(p, x, w, bits, scale, zero, a, qk, lse, gam, 0.0)
    assert torch.equal(dw, dw0) and torch.equal(ds, ds0)
