"""GPU parity of the fp32 attention backward, whose waves take every fourth (with the KL term at head_dim
128 every second) tile of a 32-row block: fewer tiles than waves, one more than a multiple, ragged last
tiles, groups of query heads.  The bars are those of the backward tests (1e-4 relative L2 per matrix
against the fp64 oracle)."""
import pytest

from test_gpu_backward import _check_backward
from test_gpu_kl_bwd import _check_kl_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [16, 64, 128])
@pytest.mark.parametrize("B,T,hq,hkv", [(1, 20, 2, 2), (2, 33, 4, 2), (1, 161, 2, 2), (1, 130, 4, 1), (8, 64, 2, 1)])
def test_fp32_backward_matches_oracle(B, T, hq, hkv, dh):
    shape = (B, T, 64, hq, hkv, dh, 32, "f32")
    _check_backward(shape)
    _check_kl_backward(shape + (0.0, 0.1))
