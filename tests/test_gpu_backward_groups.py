"""GPU parity of the bf16 backward on streamed 128-row groups at the shapes
where the groups can go wrong: blocks of 32 to 256 whose groups straddle
blocks or end inside one, odd cell columns (a pair without a right cell), one
row or column of cells, halves of 16 x 16 cells, more coarse sets than one
matrix-core chunk.  Tolerances and references as test_gpu_backward."""
import pytest

from test_gpu_backward import _case, _check, _dev, _gpu_backward

pytestmark = pytest.mark.gpu

CASES = [
    ("grp_r32_one_chunk", 1, False, "bf16", 1, 2, 32, 32, 1),
    ("grp_r32_ragged", 1, False, "bf16", 1, 2, 32 * 13, 32, 1),
    ("grp_r32_causal_p2", 1, True, "bf16", 2, 1, 32 * 9, 32, 2),
    ("grp_r64_odd_causal", 1, True, "bf16", 1, 2, 64 * 5, 64, 1),
    ("grp_r192_ragged", 1, False, "bf16", 1, 1, 192 * 5, 192, 1),
    ("grp_r192_causal", 1, True, "bf16", 1, 1, 192 * 7, 192, 1),
    ("grp_r256_causal", 1, True, "bf16", 1, 1, 256 * 5, 256, 1),
    ("grp_r64_20sets", 1, False, "bf16", 1, 1, 64 * 36, 64, 4),
    ("grp_2d_odd_cols", 2, False, "bf16", 1, 2, (40, 56), 8, 1),
    ("grp_2d_odd_cols_p2", 2, False, "bf16", 1, 1, (24, 72), 8, 2),
    ("grp_2d_row", 2, False, "bf16", 1, 1, (8, 72), 8, 1),
    ("grp_2d_column", 2, False, "bf16", 1, 1, (72, 8), 8, 1),
    ("grp_2d_r16_odd", 2, False, "bf16", 1, 1, (48, 80), 16, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_backward_groups_parity(case):
    dev = _dev()
    w, q, k, v, wk, wv, dout = _case(*case)
    _, grads = _gpu_backward(w, q, k, v, wk, wv, dout, dev)
    _check(w, q, k, v, wk, wv, dout, grads)
