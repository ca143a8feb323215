"""The sweep's attention passes of several (b_Q, b_K) sets in one launch: every triple's loss is bitwise the
forward loss with that triple's scales, for more sets than a launch takes, sets of one, two, three and more
value tensors in one call, and all seven bit-widths."""
import itertools

import pytest
import torch

from paper_2609_34866_amd import jab

from gpu_helpers import device_inputs, small

pytestmark = pytest.mark.gpu

CASES = [
    # (T, Hq, Hkv, dh, dtype, bits, every n-th triple)
    (33, 4, 4, 16, "f32", (2, 3, 4, 5, 6, 7, 8), 1),        # 343 sets of one value tensor
    (40, 4, 2, 16, "bf16", (2, 3, 4, 5, 6, 7, 8), 5),
    (70, 4, 4, 64, "f16", (2, 3, 4, 5, 6), 1),              # 25 sets of four and 25 of one
    (65, 8, 2, 128, "bf16", (2, 3, 4, 8, 5), 3),            # sets of one and two
    (64, 2, 2, 128, "bf16", (3, 4, 8), 1),                  # 9 sets of three, taken two and one
]


@pytest.mark.parametrize("case", CASES)
def test_every_triple_is_the_forward_loss(case):
    T, hq, hkv, dh, dtype, bits, nth = case
    wl = small(batch=2, seq_len=T, d_model=64, n_heads=hq, n_kv_heads=hkv, head_dim=dh, group_size=32, dtype=dtype)
    x, w = device_inputs(wl)
    p = jab.problem_of(wl)
    a = jab.attn_ref(p, x, w)
    sc = [jab.quant_init(p, w, (b, b, b)) for b in bits]
    triples = list(itertools.product(bits, repeat=3))[::-1][::nth]
    loss, per = jab.loss_sweep(p, x, w, bits, [s for s, _ in sc], [z for _, z in sc], triples, a)
    rows = (hq * dh, hkv * dh, hkv * dh)
    for i in range(0, len(triples), max(1, len(triples) // 24)):
        t = triples[i]
        cut = [0, rows[0], rows[0] + rows[1], sum(rows)]
        scale = torch.cat([sc[bits.index(b)][0][cut[m]:cut[m + 1]] for m, b in enumerate(t)])
        zero = torch.cat([sc[bits.index(b)][1][cut[m]:cut[m + 1]] for m, b in enumerate(t)])
        out = jab.loss_fwd(p, x, w, t, scale, zero, a)
        assert float(out[0]) == float(loss[i]), t
        assert torch.equal(out[3:], per[i]), t
