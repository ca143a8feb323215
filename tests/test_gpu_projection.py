"""GPU projection on every route of the GEMM dispatch (64-, 128- and 256-tiles, one launch or two, whole
and ragged sequences, values of very short ones packed, with and without the rotary embedding) against an fp32 product.

[Q|K] comes back from ``attn_ref_kl``: one rounding of the fp32 sum to the dtype (half an ulp, at most
2^-8 or 2^-11 of the value) plus the sum's own error (d terms, the two products summed in other orders).  V^T is
seen through the attention output: a softmax average of the values with probabilities rounded to the
dtype, so within a few dtype ulps of the largest value."""
import math

import pytest
import torch

from paper_2609_34866_amd import inputs, jab

from gpu_helpers import device_inputs, small

pytestmark = pytest.mark.gpu

# unit roundoff: half an ulp of a value just above a power of two
EPS = {"f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}

ROUTES = [
    # (B, T, d, Hq, Hkv, dh, dtype, rope)
    (1, 1, 64, 4, 4, 16, "f32", 0.0),             # one token, 64-tile, fp32
    (3, 47, 96, 4, 2, 64, "f32", 0.0),            # ragged 64-tile edges, three k-tiles of 32
    (8, 512, 192, 16, 8, 128, "f32", 0.0),        # 128-tile fp32
    (2, 33, 96, 8, 2, 64, "f16", 0.0),            # k-tiles of 32 (d not a multiple of 64)
    (5, 31, 64, 4, 4, 16, "bf16", 0.0),           # a single k-tile, value rows below one tile
    (3, 777, 128, 12, 12, 64, "f16", 0.0),        # 128-tiles, ragged sequences
    (3, 777, 160, 12, 12, 64, "f16", 0.0),        # ... with k-tiles of 32
    (1, 4096, 512, 32, 8, 64, "bf16", 0.0),       # 256-tiles, one launch, whole sequences
    (5, 777, 512, 32, 8, 64, "bf16", 0.0),        # 256-tiles, one launch, ragged: tiles span sequences
    (70, 45, 576, 40, 5, 64, "f16", 0.0),         # ... short sequences, ragged last tiles both ways
    (3001, 7, 512, 8, 8, 64, "bf16", 0.0),        # values over packed sequences, 18 per tile, a last tile of 13
    (3000, 3, 544, 10, 5, 64, "f16", 1e4),        # ... ragged value rows, k-tiles of 32, rotary queries and keys
    (4001, 16, 2048, 16, 16, 64, "bf16", 0.0),    # ... 8 per tile, the longest that pays
    (1001, 5, 256, 16, 16, 16, "f32", 0.0),       # ... fp32
    (2500, 1, 512, 4, 4, 64, "f32", 0.0),         # ... one token
    (500, 41, 256, 10, 10, 64, "f32", 0.0),       # ... two blocks of positions per sequence
    (1, 65, 128, 4, 1, 128, "bf16", 1e4),         # rotary 128-tile, head_dim 128
    (2, 77, 96, 8, 4, 64, "f16", 1e4),            # rotary 128-tile, head_dim 64, k-tiles of 32
    (5, 777, 512, 32, 8, 64, "bf16", 1e4),        # rotary 256-tiles, ragged, head_dim 64
    (2, 1999, 512, 16, 4, 128, "bf16", 1e4),      # rotary, head_dim 128
    (4, 1999, 512, 16, 4, 128, "f16", 1e4),       # rotary 256-tiles, head_dim 128, ragged
]


def _turn(v, theta, dh):
    half, T = dh // 2, v.shape[1]
    j = torch.arange(half, dtype=torch.float64, device=v.device)
    ang = torch.arange(T, dtype=torch.float64, device=v.device)[:, None] * theta ** (-2 * j / dh)
    cos, sin = ang.cos().float()[:, None], ang.sin().float()[:, None]
    a, b = v[..., :half], v[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


@pytest.mark.parametrize("B,T,d,hq,hkv,dh,dtype,rope", ROUTES)
def test_projection_routes(B, T, d, hq, hkv, dh, dtype, rope):
    wl = small(batch=B, seq_len=T, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=dh, group_size=32,
               dtype=dtype, rope_theta=rope)
    x, w = device_inputs(wl)
    p = jab.problem_of(wl)
    a, qk, _ = jab.attn_ref_kl(p, x, w)
    y = (x.double().reshape(B * T, d) @ w.double().t()).float().reshape(B, T, -1)
    nq, nk = hq * dh, hkv * dh
    q, k = y[..., :nq].reshape(B, T, hq, dh), y[..., nq:nq + nk].reshape(B, T, hkv, dh)
    if rope:
        q, k = _turn(q, rope, dh), _turn(k, rope, dh)
    want = torch.cat([q.reshape(B, T, nq), k.reshape(B, T, nk)], -1).reshape(B * T, nq + nk)
    eps = EPS[dtype]
    # sum error: at most d 2^-23 of the sum of the products' magnitudes, whose root is about the value's
    # scale; a turned pair adds its partner's
    scale = want.abs().amax()
    err = (qk.float() - want).abs()
    assert float((err - (eps * want.abs() + scale * 2.0 ** -18)).amax()) <= 0.0
    # the attention output from the projection as stored
    qf = qk.float().reshape(B, T, -1)
    q, k = qf[..., :nq].reshape(B, T, hq, dh), qf[..., nq:].reshape(B, T, hkv, dh)
    v = y[..., nq + nk:].to(wl.torch_dtype).float().reshape(B, T, hkv, dh)
    mask = torch.ones(T, T, dtype=torch.bool, device=x.device).triu(1)
    for b in range(B):
        kh = k[b].permute(1, 2, 0).repeat_interleave(hq // hkv, 0).contiguous()
        vh = v[b].permute(1, 0, 2).repeat_interleave(hq // hkv, 0).contiguous()
        z = torch.bmm(q[b].permute(1, 0, 2).contiguous(), kh) / math.sqrt(dh)
        o = torch.bmm(torch.softmax(z.masked_fill(mask, -math.inf), -1), vh)
        got = a[b].reshape(T, hq, dh).permute(1, 0, 2)
        # P rounded to the dtype (half an ulp each), the values' own rounding where the two fp32 sums
        # round apart (an ulp), the exponentials' argument error (2^-18 at |z| up to 2^5)
        assert float((got - o).abs().amax()) <= (2 * eps + 2.0 ** -16) * float(vh.abs().amax()), b


def test_projection_split_batches_agree():
    """The same tokens as one batch and as single sequences (other tiles, other routes): the [Q|K] rows
    and the 16-bit products' order are the same on every route, so the bits are too."""
    wl = small(batch=5, seq_len=777, d_model=512, n_heads=32, n_kv_heads=8, head_dim=64, group_size=32, dtype="bf16")
    x, w = device_inputs(wl)
    qk = jab.attn_ref_kl(jab.problem_of(wl), x, w)[1]
    for b in (0, 4):
        one = jab.attn_ref_kl(jab.problem_of(wl, batch=1), x[b:b + 1].contiguous(), w)[1]
        assert torch.equal(one, qk[b * 777:(b + 1) * 777])
