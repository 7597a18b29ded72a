"""Units of the 1D bf16 streaming coarsening with more than 16 coarse sets:
the widest whose rounds keep the resident waves busy.  The addresses of the
chosen units are emulated on the CPU; on the GPU a plan with units of one
block (every set wider than a block left as partial sums) against the oracle."""
import pytest
import torch

import fma_inputs
import issue_emulation as emu
import oracle
import paper_2310_11960_amd as F
from test_gpu_parity import TOL, _dev, _np, rel_err

CASES = [  # batch, heads, n, block, rank, unit
    (8, 12, 16384, 128, 4, 512), (8, 9, 4096, 64, 4, 64), (1, 2, 16384, 128, 4, 128), (8, 12, 16384, 128, 2, 1024)]   # at most 16 sets: the widest that fills the chip once


@pytest.mark.parametrize("case", CASES, ids=str)
def test_unit_rule_and_addresses(case):
    B, H, n, r, p, unit = case
    op = F.FMA(ndim=1, batch=B, heads=H, seq_len=n, block=r, rank=p, dtype=torch.bfloat16)
    P = F.fma_plan_params(op.handle)
    assert P["chunk"] == unit
    emu.check_coarsen1d_stream(P)


@pytest.mark.gpu
def test_narrow_units_parity():
    dev = _dev()
    B, H, n, r, p, _ = CASES[1]
    w = fma_inputs.custom("units_of_a_block", 1, False, "bf16", B, H, n, block=r, seed=41, rank=p)
    q, k, v, wk, wv = fma_inputs.make_inputs(w)
    op = F.FMA(ndim=1, batch=B, heads=H, seq_len=n, block=r, rank=p, dtype=torch.bfloat16)
    kb, vb = op.coarse_views(op.coarsen(k.to(dev), v.to(dev), wk.to(dev), wv.to(dev)))
    torch.cuda.synchronize()
    for b, h in ((0, 0), (3, 5), (7, 8)):
        for got, x, wt in ((kb, k, wk), (vb, v, wv)):
            ref = oracle.coarsen_1d(_np(x[b, h]), r, _np(wt[h]), rank=p)
            assert rel_err(_np(got[b, h].cpu()), ref) <= TOL["bf16"], (b, h)
