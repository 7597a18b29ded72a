"""GPU parity of maps and sequences without a coarse level (at most two cells
per side, at most two blocks): no interaction list, so the normalisation and
the rank change nothing, and every call runs whatever list slots per level
its plan works out.  References and tolerances as test_gpu_parity and
test_gpu_backward."""
import zlib

import pytest
import torch

import fma_inputs
from test_gpu_backward import _case, _check, _gpu_backward
from test_gpu_parity import _check_slices, _dev, _run

pytestmark = pytest.mark.gpu

MAPS = [(r, cells, rank, per_level) for r in (8, 16) for cells in ((1, 1), (1, 2), (2, 2)) for rank in (1, 2)
        for per_level in (False, True)]


@pytest.mark.parametrize("dtype,head_dim", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("r,cells,rank,per_level", MAPS)
def test_map_without_levels(r, cells, rank, per_level, dtype, head_dim):
    dev = _dev()
    name = "nolev_%dx%d_r%d_p%d_%s_d%d%s" % (*cells, r, rank, dtype, head_dim, "_level" if per_level else "")
    w = fma_inputs.custom(name, 2, False, dtype, 1, 2, side=r * cells[1], height=r * cells[0], block=r, rank=rank,
                          head_dim=head_dim, seed=zlib.crc32(name.encode()) % 1000)
    q, k, v, wk, wv = fma_inputs.make_inputs(w)
    assert wk.numel() == 0
    _, out = _run(w, q, k, v, wk, wv, dev, per_level=per_level)
    _check_slices(w, q, k, v, wk, wv, out, per_level=per_level, case=name)


@pytest.mark.parametrize("r,blocks", [(32, 2), (64, 1), (128, 2), (192, 2), (256, 1)])
@pytest.mark.parametrize("rank,per_level", [(1, True), (2, True), (10, True), (3, False)])
def test_sequence_without_levels(r, blocks, rank, per_level):
    dev = _dev()
    name = "nolev_n%d_r%d_p%d%s" % (r * blocks, r, rank, "_level" if per_level else "")
    w = fma_inputs.custom(name, 1, True, "bf16", 1, 2, n=r * blocks, block=r, rank=rank,
                          seed=zlib.crc32(name.encode()) % 1000)
    q, k, v, wk, wv = fma_inputs.make_inputs(w)
    _, out = _run(w, q, k, v, wk, wv, dev, per_level=per_level)
    _check_slices(w, q, k, v, wk, wv, out, per_level=per_level, case=name)


@pytest.mark.parametrize("r,cells,rank", [(8, (2, 2), 2), (8, (1, 2), 3), (16, (2, 1), 2), (8, (2, 2), 1)])
def test_map_without_levels_backward(r, cells, rank):
    dev = _dev()
    w, q, k, v, wk, wv, dout = _case("nolev_bwd_r%d_%dx%d_p%d" % (r, *cells, rank), 2, False, "bf16", 1, 2,
                                     (r * cells[0], r * cells[1]), r, rank)
    _, grads = _gpu_backward(w, q, k, v, wk, wv, dout, dev, per_level=True)
    assert torch.isfinite(grads[0].float()).all()
    _check(w, q, k, v, wk, wv, dout, grads, per_level=True)
