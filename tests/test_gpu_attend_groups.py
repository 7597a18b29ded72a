"""GPU parity of the bf16 attention on groups of 128 queries at the shapes
where the groups can go wrong: one chunk, groups that straddle blocks or end
inside one, 1D blocks of 32 to 256 at head dims 32, 64 and 128, odd cell
columns, one row or column of cells, more list rows than one tile, per-level
lists of both cells of a pair, and scores far above the first piece's.
References and tolerances as test_gpu_parity."""
import zlib

import pytest
import torch

import fma_inputs
from test_gpu_parity import _check_slices, _dev, _run

pytestmark = pytest.mark.gpu

CASES = [
    # name, ndim, causal, B, H, n or (rows, columns), r, rank, per_level, head_dim
    ("att_r32_one_chunk", 1, False, 1, 2, 32, 32, 1, False, 64),
    ("att_r32_ragged_causal", 1, True, 1, 3, 32 * 13, 32, 1, False, 64),
    ("att_r32_p4", 1, False, 1, 1, 32 * 37, 32, 4, False, 64),
    ("att_r32_level", 1, True, 1, 2, 32 * 21, 32, 1, True, 64),
    ("att_r64_odd", 1, False, 1, 2, 64 * 5, 64, 1, False, 64),
    ("att_r192_causal", 1, True, 1, 2, 192 * 7, 192, 1, False, 64),
    ("att_r128_small", 1, False, 1, 2, 128 * 9, 128, 2, False, 64),
    ("att_r256_level", 1, False, 1, 1, 256 * 5, 256, 1, True, 64),
    ("att_d128_r32", 1, False, 1, 2, 32 * 9, 32, 1, False, 128),
    ("att_d128_r192_causal", 1, True, 1, 1, 192 * 5, 192, 2, False, 128),
    ("att_d128_level", 1, True, 1, 2, 64 * 11, 64, 1, True, 128),
    ("att_d32_r256", 1, True, 1, 2, 256 * 5, 256, 1, False, 32),
    ("att_d32_2d", 2, False, 1, 2, (24, 40), 8, 1, False, 32),
    ("att_d128_2d_odd_p2", 2, False, 1, 1, (40, 72), 8, 2, False, 128),
    ("att_d128_2d_r16_level", 2, False, 1, 1, (48, 80), 16, 1, True, 128),
    ("att_2d_odd_cols", 2, False, 1, 2, (40, 56), 8, 1, False, 64),
    ("att_2d_odd_level", 2, False, 1, 2, (40, 56), 8, 1, True, 64),
    ("att_2d_row", 2, False, 1, 1, (8, 72), 8, 1, False, 64),
    ("att_2d_column_level", 2, False, 1, 1, (72, 8), 8, 1, True, 64),
    ("att_2d_p4", 2, False, 1, 1, (64, 72), 8, 4, False, 64),
    ("att_2d_r16_odd", 2, False, 1, 1, (48, 80), 16, 2, False, 64),
]


def _workload(case):
    name, ndim, causal, B, H, size, r, p, per_level, d = case
    kw = dict(n=size) if ndim == 1 else dict(height=size[0], side=size[1])
    return fma_inputs.custom(name, ndim, causal, "bf16", B, H, block=r, seed=zlib.crc32(name.encode()) % 1000, rank=p,
                             head_dim=d, **kw)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_attend_groups_parity(case):
    dev = _dev()
    w = _workload(case)
    q, k, v, wk, wv = fma_inputs.make_inputs(w)
    _, out = _run(w, q, k, v, wk, wv, dev, per_level=case[8])
    _check_slices(w, q, k, v, wk, wv, out, per_level=case[8], case=w.name)


@pytest.mark.parametrize("case", [c for c in CASES if c[0] in (
    "att_r32_ragged_causal", "att_r192_causal", "att_d128_r32", "att_d32_r256", "att_d128_2d_odd_p2",
    "att_2d_odd_level")], ids=lambda c: c[0])
def test_attend_groups_score_jumps(case):
    """Every fourth key of the second half scores up to 784 log2 units above
    the first piece (exact integer scores, fma_inputs.make_peaked_inputs)."""
    dev = _dev()
    w = _workload(case)
    q, k, v, wk, wv = fma_inputs.make_peaked_inputs(w)
    idx = torch.arange(w.n // 2, w.n, 4)
    q[..., 0] = 2
    k[:, :, idx, :] = 0
    k[:, :, idx, 0] = 400
    scale = fma_inputs.PEAKED_SCALE
    _, out = _run(w, q, k, v, wk, wv, dev, per_level=case[8], scale=scale)
    assert torch.isfinite(out.float()).all()
    _check_slices(w, q, k, v, wk, wv, out, per_level=case[8], scale=scale, case=w.name + "_jump")
