"""GPU parity of the fp32 attention whose keys are split over four waves (at
most 256 pieces of 32 queries) at its edges: fewer tiles than waves, blocks
below 32 queries, 256 pieces and one block more, more list rows than one round
of tiles, ragged maps.  References and tolerances as test_gpu_parity."""
import zlib

import pytest
import torch

import fma_inputs
from test_gpu_parity import _check_slices, _dev, _run

pytestmark = pytest.mark.gpu

CASES = [
    # name, ndim, causal, B, H, n or (rows, columns), r, rank, head_dim
    ("split_r16_causal", 1, True, 1, 2, 16 * 9, 16, 1, 64),
    ("split_r32", 1, False, 1, 1, 32 * 3, 32, 1, 64),
    ("split_r64_causal_odd", 1, True, 1, 3, 64 * 7, 64, 1, 64),
    ("split_r64_p5", 1, False, 1, 1, 64 * 33, 64, 5, 64),
    ("split_256_pieces", 1, True, 2, 4, 64 * 16, 64, 1, 64),
    ("split_258_pieces", 1, False, 1, 1, 64 * 129, 64, 1, 64),
    ("split_r256_causal", 1, True, 1, 2, 256 * 5, 256, 1, 64),
    ("split_r192", 1, False, 1, 1, 192 * 5, 192, 2, 32),
    ("split_2d_ragged", 2, False, 1, 2, (24, 40), 8, 1, 64),
    ("split_2d_r4_p3", 2, False, 1, 1, (36, 20), 4, 3, 64),
    ("split_2d_r16_d32", 2, False, 1, 1, (48, 80), 16, 1, 32),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_attend_split_parity(case):
    dev = _dev()
    name, ndim, causal, B, H, size, r, p, d = case
    kw = dict(n=size) if ndim == 1 else dict(height=size[0], side=size[1])
    w = fma_inputs.custom(name, ndim, causal, "f32", B, H, block=r, seed=zlib.crc32(name.encode()) % 1000, rank=p,
                          head_dim=d, **kw)
    q, k, v, wk, wv = fma_inputs.make_inputs(w)
    _, out = _run(w, q, k, v, wk, wv, dev)
    _check_slices(w, q, k, v, wk, wv, out, case=w.name)
    assert torch.isfinite(out).all()
