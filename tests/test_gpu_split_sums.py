"""GPU sums that are split over workgroups: the weight gradient's parts of K (two to sixteen, 64- and
128-tiles), and the loss and weight-error reductions that the last of their workgroups finishes.

The gradient bars are test_gpu_backward's (2e-2 for the 16-bit dtypes, 1e-4 for fp32, relative L2 per
matrix against the fp64 oracle)."""
import numpy as np
import pytest
import torch

from paper_2609_34866_amd import inputs, jab

from gpu_helpers import device_inputs, small
from test_gpu_backward import _check_backward

pytestmark = pytest.mark.gpu

PARTS = [
    # (B, T, d, Hq, Hkv, dh, g, dtype): K = B T rounded up to 64
    (2, 520, 128, 4, 2, 64, 32, "f16"),       # two parts of 17 k-tiles of 64 (8 and 9)
    (3, 700, 96, 4, 4, 64, 32, "bf16"),       # four parts, output columns below one tile
    (1, 545, 128, 4, 4, 16, 32, "f32"),       # two parts of k-tiles of 32, fp32
    (40, 430, 64, 2, 2, 64, 32, "f16"),       # sixteen parts
]


@pytest.mark.parametrize("shape", PARTS)
def test_weight_gradient_parts_match_oracle(shape):
    _check_backward(shape)


@pytest.mark.parametrize("B,T", [(1, 1), (1, 33), (63, 8), (64, 8), (65, 8), (3, 1100), (200, 40), (256, 2), (257, 2),
                                 (513, 1), (1100, 1)])
def test_loss_reduction_is_the_sum_of_its_sequences(B, T):
    """out against the per-sequence sums it returns, and those against single-sequence calls, for batches
    around a wavefront and partial counts around the unrolled loops; the same bits on every call.  From 257
    sequences on the two sets of the KL call take two launches, the loss alone one up to 512: equal bits."""
    wl = small(batch=B, seq_len=T, d_model=64, n_heads=4, n_kv_heads=4, head_dim=16, group_size=32, dtype="bf16")
    x, w = device_inputs(wl)
    p, bits = jab.problem_of(wl), (3, 4, 2)
    scale, zero = jab.quant_init(p, w, bits)
    a, qk, lse = jab.attn_ref_kl(p, x, w)
    out = jab.loss_fwd_kl(p, x, w, bits, scale, zero, a, qk, lse)
    for _ in range(3):
        assert torch.equal(jab.loss_fwd_kl(p, x, w, bits, scale, zero, a, qk, lse), out)
    assert torch.equal(jab.loss_fwd(p, x, w, bits, scale, zero, a), out[:3 + B])
    o = out.cpu().numpy()
    n = B * T * 64
    np.testing.assert_allclose(o[0], o[3:3 + B].sum(), rtol=1e-13)         # fp64 sums of up to 1100 terms
    np.testing.assert_allclose(o[1], o[0] / n, rtol=1e-14)
    np.testing.assert_allclose(o[2], float((a.double() ** 2).sum()), rtol=1e-6)   # fp32 squares per tile
    np.testing.assert_allclose(o[3 + B], o[6 + B:].sum(), rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(o[4 + B], o[3 + B] / B, rtol=1e-14)
    one = jab.problem_of(wl, batch=1)
    for b in {0, B // 2, B - 1}:
        a1 = jab.attn_ref(one, x[b:b + 1].contiguous(), w)
        l1 = jab.loss_fwd(one, x[b:b + 1].contiguous(), w, bits, scale, zero, a1)
        assert float(l1[0]) == o[3 + b], b
    loss, per = jab.loss_sweep(p, x, w, (3, 4), [jab.quant_init(p, w, (c, c, c))[0] for c in (3, 4)],
                               [jab.quant_init(p, w, (c, c, c))[1] for c in (3, 4)], [(3, 3, 4), (4, 3, 3)], a)
    np.testing.assert_allclose(loss.cpu().numpy(), per.cpu().numpy().sum(1), rtol=1e-13)


@pytest.mark.parametrize("rows,d", [(1, 64), (3, 128), (255 * 4, 2048), (256 * 4 + 5, 2048)])
def test_weight_error_reduction(rows, d):
    """werr over one quantizer workgroup up to more than the reduction's workgroups, against fp64."""
    p = jab.problem(1, 32, d, rows, rows, 16, 64, torch.bfloat16)
    w = torch.randn((3 * rows * 16, d), device="cuda").to(torch.bfloat16)
    scale, zero = jab.quant_init(p, w, (3, 2, 4))
    q = jab.quantize(p, w, (3, 2, 4), scale, zero)
    err, ref = (q["w_hat"].double() - w.double()) ** 2, w.double() ** 2
    want = torch.stack([torch.stack([t[m * rows * 16:(m + 1) * rows * 16].sum() for t in (err, ref)]) for m in range(3)])
    np.testing.assert_allclose(q["werr"].cpu().numpy(), want.cpu().numpy(), rtol=1e-12)
    assert torch.equal(jab.quantize(p, w, (3, 2, 4), scale, zero)["werr"], q["werr"])
