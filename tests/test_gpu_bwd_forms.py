"""GPU parity of every form of the dK/dV pass of the 16-bit backward (head_dim 64 and 128): one, two or
four key slices per workgroup, one workgroup per key block, and the paired form, chosen by the number of
key blocks; ragged query tiles, steps that a way has no tile for.  The bars are
those of the backward tests (relative L2 per matrix against the fp64 oracle, 2e-2)."""
import pytest
import torch

from paper_2609_34866_amd import jab

from gpu_helpers import device_inputs
from test_gpu_backward import _check_backward, _wl
from test_gpu_kl_bwd import _check_kl_backward

pytestmark = pytest.mark.gpu

FORMS = [
    # (B, T, d, Hq, Hkv, dh, g, dtype)
    (1, 1, 64, 4, 2, 64, 32, "bf16"),         # one slice, one tile for four ways
    (1, 300, 96, 12, 1, 64, 32, "bf16"),      # one slice, a group of twelve
    (33, 129, 64, 8, 2, 64, 32, "f16"),       # two slices, a last block of one key
    (130, 70, 64, 2, 2, 64, 32, "f16"),       # four slices
    (1, 67, 64, 12, 1, 128, 32, "f16"),       # two slices, a group of twelve
    (97, 65, 64, 2, 2, 128, 32, "bf16"),      # four slices
    (193, 40, 64, 2, 2, 128, 32, "bf16"),     # paired
    (513, 40, 64, 2, 2, 64, 32, "f16"),       # paired at head_dim 64 (with the KL term from 257 pairs on)
]


@pytest.mark.parametrize("ds_limit", [8 << 30, 0])
@pytest.mark.parametrize("shape", FORMS)
def test_dkdv_forms_match_oracle(shape, ds_limit):
    jab.set_bwd_ds_limit(ds_limit)
    try:
        _check_backward(shape)
        _check_kl_backward(shape + (10000.0 if shape[1] == 67 else 0.0, 0.1))
    finally:
        jab.set_bwd_ds_limit(8 << 30)


# the paired form of the KL term (head_dim 64) and its two slices
@pytest.mark.parametrize("shape", [(128, 33, 64, 2, 2, 64, 32, "bf16", 0.0, 0.1), (65, 129, 64, 4, 2, 64, 32, "f16", 0.0, 0.1)])
def test_dkdv_forms_with_the_kl_term_match_oracle(shape):
    _check_kl_backward(shape)


@pytest.mark.parametrize("shape", FORMS + [(2, 1000, 64, 4, 4, 64, 32, "bf16"), (128, 40, 64, 2, 2, 64, 32, "f16")])
def test_lambda_zero_is_the_plain_backward_in_every_form(shape):
    wl = _wl(*shape)
    x, w = device_inputs(wl)
    p, bits = jab.problem_of(wl), (3, 4, 2)
    scale, zero = jab.quant_init(p, w, bits)
    a, qk, lse = jab.attn_ref_kl(p, x, w)
    gam = jab.lsq_gscale(bits, wl.group_size)
    _, dw, ds = jab.loss_bwd(p, x, w, bits, scale, zero, a, gam)
    _, dw0, ds0 = jab.loss_bwd_kl(p, x, w, bits, scale, zero, a, qk, lse, gam, 0.0)
    assert torch.equal(dw, dw0) and torch.equal(ds, ds0)
