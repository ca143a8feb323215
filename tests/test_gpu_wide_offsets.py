"""GPU calls whose tensors pass 2^32 bytes from a kernel's base address: the rows of a head's transposed
values (many short sequences: each is padded to 32 tokens), a sequence's keys (many heads).  A 32-bit
offset that wraps reads other rows without an error.  References in fp32 from the tensors as stored; the
bounds are those of the projection tests (roundings of the values and of the probabilities)."""
import math

import pytest
import torch

from paper_2609_34866_amd import jab

pytestmark = pytest.mark.gpu

EPS = {torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11}


def _inputs(rows, B, T, d, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    x = torch.randn((B, T, d), generator=gen, device="cuda").to(dtype)
    w = (torch.randn((rows, d), generator=gen, device="cuda") * 0.1).to(dtype)
    return x, w


# one token per sequence: a query's output is its value.  the last row of a
# head starts 64 B (head_dim - 1) bytes after its first, just past 2^32
@pytest.mark.parametrize("dh,hq,hkv,B,dtype", [(128, 1, 1, 528500, torch.bfloat16), (64, 2, 1, 1065300, torch.float16),
                                               (128, 4, 1, 528500, torch.float16)])
def test_value_rows_past_4_gib(dh, hq, hkv, B, dtype):
    d = 32
    p = jab.problem(B, 1, d, hq, hkv, dh, 32, dtype)
    x, w = _inputs(p.rows, B, 1, d, dtype)
    a = jab.attn_ref(p, x, w)
    v = x.reshape(B, d).float() @ w[-dh:].float().t()
    eps = EPS[dtype]
    for h in range(hq):
        err = (a[:, 0, h * dh:(h + 1) * dh] - v).abs()
        assert float((err - (eps * v.abs() + v.abs().amax() * 2.0 ** -18)).amax()) <= 0.0, h
    widths = (2, 4)
    sets = [jab.quant_init(p, w, (b, b, b)) for b in widths]
    triples = [(4, 2, 2), (4, 2, 4), (4, 4, 4)]
    total, per = jab.loss_sweep(p, x, w, widths, [s for s, _ in sets], [z for _, z in sets], triples, a)
    out = jab.loss_fwd(p, x, w, (4, 4, 4), *sets[1], a)
    assert float(out[0]) == float(total[2]) and torch.equal(out[3:], per[2])
    w_hat = jab.quantize(p, w, (4, 4, 4), *sets[1])["w_hat"][-dh:].to(dtype).float()
    v_hat = (x.reshape(B, d).float() @ w_hat.t()).to(dtype).float()
    want = hq * (v_hat - v.to(dtype).float()).double().square().sum(1)
    # each difference of two rounded values moves by their ulps where the fp32 sums round apart: the sums
    # of all sequences agree far closer than one sequence's
    assert abs(float(out[0]) - float(want.sum())) <= 1e-3 * float(want.sum())
    assert float((out[3:] - want).abs().amax()) <= 0.1 * float(want.amax())


def test_keys_past_4_gib():
    """512 heads of 128 in one sequence of 16512 tokens: 4.3 GB of [Q | K] rows."""
    T, heads, dh, d, dtype = 16512, 512, 128, 32, torch.bfloat16
    p = jab.problem(1, T, d, heads, heads, dh, 32, dtype)
    x, w = _inputs(p.rows, 1, T, d, dtype)
    a, qk, lse = jab.attn_ref_kl(p, x, w)
    mask = torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)
    for h in (0, 300, heads - 1):
        q = qk[:, h * dh:(h + 1) * dh].float()
        k = qk[:, (heads + h) * dh:(heads + h + 1) * dh].float()
        v = (x[0].float() @ w[(2 * heads + h) * dh:(2 * heads + h + 1) * dh].float().t()).to(dtype).float()
        z = ((q @ k.t().contiguous()) / math.sqrt(dh)).masked_fill_(mask, -math.inf)
        assert float((lse[0, h] * math.log(2.0) - torch.logsumexp(z, -1)).abs().amax()) <= 1e-3, h
        o = torch.softmax(z, -1) @ v
        got = a[0, :, h * dh:(h + 1) * dh]
        assert float((got - o).abs().amax()) <= (2 * EPS[dtype] + 2.0 ** -16) * float(v.abs().amax()), h
        del z, o
    # the float point's map equals the teacher's: both terms are exactly 0, and its rows sum to 1
    out = jab.loss_fwd_kl(p, x, w, (0, 0, 0), None, None, a, qk, lse)
    assert float(out[0]) == 0.0 and float(out[4]) == 0.0
    assert abs(float(out[6])) <= 1e-4 * heads * T


# the weight gradient contracts over the tokens, so its operands' rows are as long as the batch has tokens:
# 64 rows of them pass 2^32 bytes
@pytest.mark.parametrize("dtype,hq,dh,B,bar", [(torch.float32, 2, 16, 533300, 1e-3), (torch.bfloat16, 1, 64, 1065300, 2e-2)])
def test_weight_gradient_of_many_tokens(dtype, hq, dh, B, bar):
    """bar: the running fp32 sums of a part's million tokens (2^-24 per step, as its square root: 6e-5); in
    16 bits the backward tests' 2e-2 for gradients."""
    T, d = 32, 32
    p = jab.problem(B, T, d, hq, 1, dh, 32, dtype)
    x, w = _inputs(p.rows, B, T, d, dtype)
    bits = (3, 3, 3)
    scale, zero = jab.quant_init(p, w, bits)
    a = jab.attn_ref(p, x, w)
    _, dw, _ = jab.loss_bwd(p, x, w, bits, scale, zero, a, jab.lsq_gscale(bits, 32))
    w_hat = jab.quantize(p, w, bits, scale, zero)["w_hat"].to(dtype).double()
    want = torch.zeros_like(w_hat)
    mask = torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)
    for b0 in range(0, B, 32768):
        xb = x[b0:b0 + 32768].double()
        *qs, k, v = ((xb @ m.t().contiguous()) for m in w_hat.split(dh))
        kt, vt = k.transpose(1, 2).contiguous(), v.transpose(1, 2).contiguous()
        dq, dk, dv = [], 0.0, 0.0
        for h, q in enumerate(qs):
            z = torch.bmm(q, kt) / math.sqrt(dh)
            prob = torch.softmax(z.masked_fill_(mask, -math.inf), -1)
            g = (torch.bmm(prob, v) - a[b0:b0 + 32768, :, h * dh:(h + 1) * dh]) * (2.0 / (B * T * hq * dh))
            dp = torch.bmm(g, vt)
            dz = prob * (dp - (dp * prob).sum(-1, keepdim=True)) / math.sqrt(dh)
            dq.append(torch.bmm(dz, k))
            dk = dk + torch.bmm(dz.transpose(1, 2).contiguous(), q)
            dv = dv + torch.bmm(prob.transpose(1, 2).contiguous(), g)
        dy = torch.cat(dq + [dk, dv], -1)
        want += dy.reshape(-1, p.rows).t().contiguous() @ xb.reshape(-1, d)
    for m, (got, ref) in enumerate(zip(dw.double().split(dh), want.split(dh))):
        assert float((got - ref).norm()) <= bar * float(ref.norm()), m


def test_projection_of_wide_rows():
    """17.1 M input channels: the 64 rows of the activations pass 2^32 bytes."""
    d, T, dtype = 17_100_000 // 32 * 32, 64, torch.float32
    p = jab.problem(1, T, d, 1, 1, 16, 32, dtype)
    x, w = _inputs(p.rows, 1, T, d, dtype)
    y = jab.project(p, x, w)[0].double()
    want = torch.zeros_like(y)
    for k in range(0, d, 1 << 20):
        want += x[0, :, k:k + (1 << 20)].double() @ w[:, k:k + (1 << 20)].double().t().contiguous()
    # 17 M running fp32 sums: 2^-24 per step as its square root, 2.5e-4
    assert float((y - want).norm()) <= 2e-3 * float(want.norm())
