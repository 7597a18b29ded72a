"""The softmax scale may be negative: scale -t with queries q is scale t with
queries -q.  Every product of the two calls differs in sign at most: the
outputs are equal, bit for bit, the gradients of k, v and the weights agree and
dq changes sign.

The gradients' matrix products add terms whose signs differ between the two
calls, and the matrix cores' alignment of a sum is not symmetric in the sign,
so 32-bit sums may differ in their last bits, and a bf16 result or rounded
weight by one unit, 2^-8 of itself, where such a sum lies on a boundary.  The
bound is a unit of the largest value and as much again for flipped weights,
2^-7 of the maximum; 32-bit calls keep the parity tests' 1e-5."""
import pytest
import torch

import paper_2310_11960_amd as F

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}

# ndim, causal, dtype, n or (rows, columns), r, head_dim, rank, per_level
FORWARD = [
    (1, True, "bf16", 64 * 7, 64, 128, 1, False), (1, False, "bf16", 32 * 13, 32, 64, 1, False),
    (1, True, "bf16", 32 * 13, 32, 64, 1, True), (1, False, "bf16", 256 * 5, 256, 32, 2, False),
    (2, False, "bf16", (24, 40), 8, 128, 1, False), (2, False, "bf16", (48, 80), 16, 32, 1, True),
    (1, True, "bf16", 128 * 9, 128, 64, 1, False), (1, False, "bf16", 192 * 5, 192, 64, 1, False),
    (2, False, "bf16", (40, 56), 8, 64, 1, False), (2, False, "bf16", (40, 48), 8, 64, 2, True),
    (1, True, "bf16", 16 * 9, 16, 64, 1, False), (2, False, "bf16", (20, 36), 4, 64, 1, False),
    (1, True, "f32", 64 * 7, 64, 64, 1, False), (2, False, "f32", (24, 40), 8, 64, 1, False),
    (1, False, "f32", 64 * 140, 64, 64, 1, False),
]
BACKWARD = [
    (1, True, "bf16", 128 * 9, 128, 64, 1, False), (1, False, "bf16", 32 * 13, 32, 64, 1, False),
    (1, True, "bf16", 64 * 9, 64, 64, 2, False), (2, False, "bf16", (40, 56), 8, 64, 1, False),
    (2, False, "bf16", (48, 80), 16, 64, 1, False), (1, True, "bf16", 16 * 9, 16, 64, 1, False),
    (1, True, "bf16", 64 * 9, 64, 64, 1, True), (2, False, "bf16", (40, 56), 8, 64, 2, True),
    (1, True, "f32", 64 * 9, 64, 64, 1, False), (2, False, "f32", (24, 40), 8, 64, 1, True),
]


def _ids(c):
    return "%dd_%s_%s_%s_r%d_d%d_p%d%s" % (c[0], "causal" if c[1] else "bidi", c[2],
                                          "%dx%d" % c[3] if c[0] == 2 else c[3], c[4], c[5], c[6], "_level" if c[7] else "")


def _setup(case, linear=False, seed=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ndim, causal, dt, size, r, d, rank, per_level = case
    n, side = (size, 0) if ndim == 1 else (size[0] * size[1], size[1])
    ops = [F.FMA(ndim=ndim, batch=1, heads=2, seq_len=n, block=r, causal=causal, dtype=DT[dt], side=side, head_dim=d,
                 rank=rank, softmax_scale=s * d ** -0.5, linear=linear,
                 norm=F.FMA_NORM_PER_LEVEL if per_level else F.FMA_NORM_JOINT) for s in (-1, 1)]
    g = torch.Generator().manual_seed(seed)
    x = [torch.randn((1, 2, n, d), generator=g).to(DT[dt]).cuda() for _ in range(4)]
    w = [(torch.randn((2, ops[0].weights_len), generator=g) / r ** 0.5).cuda() for _ in range(3)]
    return ops, x, w


def _same(a, b, what, bound=0.0):
    assert torch.isfinite(a.float()).all(), what
    err = float((a.float() - b.float()).abs().max()) / max(float(b.float().abs().max()), 1e-30)
    assert err <= bound, (what, err)


BOUND = {"bf16": 2.0 ** -7, "f32": 1e-5}


@pytest.mark.parametrize("case", FORWARD, ids=_ids)
def test_forward_negative_scale(case):
    ops, (q, k, v, _), (wk, wv, _) = _setup(case)
    out = [op.forward(s * q, k, v, wk, wv) for op, s in zip(ops, (1, -1))]
    torch.cuda.synchronize()
    _same(out[0], out[1], "out")


@pytest.mark.parametrize("case", BACKWARD, ids=_ids)
def test_backward_negative_scale(case):
    ops, (q, k, v, do), (wk, wv, _) = _setup(case)
    out = ops[1].forward(-q, k, v, wk, wv)
    g = [op.backward(s * q, k, v, wk, wv, out, do) for op, s in zip(ops, (1, -1))]
    torch.cuda.synchronize()
    _same(g[0][0], -g[1][0], "dq", BOUND[case[2]])
    for x, name in zip(range(1, 5), ("dk", "dv", "dwk", "dwv")):
        _same(g[0][x], g[1][x], name, BOUND[case[2]])


@pytest.mark.parametrize("dt,size,r", [("bf16", 64 * 9, 64), ("f32", 64 * 9, 64), ("bf16", (40, 56), 8), ("bf16", 16 * 9, 16)])
def test_linear_negative_scale(dt, size, r):
    ops, (q, k, v, do), (wk, wv, wq) = _setup((2 if isinstance(size, tuple) else 1, False, dt, size, r, 64, 1, False), True)
    # -q with the same wq negates the coarse queries as well
    out = [op.forward_linear(s * q, k, v, wq, wk, wv) for op, s in zip(ops, (1, -1))]
    g = [op.backward_linear(s * q, k, v, wk, wv, wq, out[1], do) for op, s in zip(ops, (1, -1))]
    torch.cuda.synchronize()
    _same(out[0], out[1], "out")
    _same(g[0][0], -g[1][0], "dq", BOUND[dt])
    for x, name in zip(range(1, 6), ("dk", "dv", "dwk", "dwv", "dwq")):
        _same(g[0][x], g[1][x], name, BOUND[dt])
