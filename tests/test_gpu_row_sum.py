"""The row sum of the bf16 attention at head dims 32 and 128 and blocks of 32
adds the fp32 weights, not their bf16 roundings: one key of weight 1 carries
the values, 63 keys of weight w (halfway between two bf16 numbers) and value
0 only enter the sum.  1 / (1 + 63 w) is a bf16 number, 230 / 2048; with w
rounded to bf16 the result rounds to the next one."""
import math

import pytest
import torch

import paper_2310_11960_amd as F

pytestmark = pytest.mark.gpu

OUT = 230 / 2048
W = (1 / OUT - 1) / 63


def test_weights_round_away():
    """(The inputs do what the docstring says.)"""
    w16 = float(torch.tensor(W).bfloat16())
    assert float(torch.tensor(1 / (1 + 63 * w16)).bfloat16()) == 231 / 2048
    assert float(torch.tensor(1 / (1 + 63 * W)).bfloat16()) == OUT


@pytest.mark.parametrize("ndim,r,head_dim", [(1, 64, 128), (1, 64, 32), (1, 32, 64), (2, 8, 128), (2, 8, 32)])
def test_row_sum_adds_fp32_weights(ndim, r, head_dim):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    op = F.FMA(ndim=ndim, batch=1, heads=1, seq_len=64, block=r, dtype=torch.bfloat16, side=8 if ndim == 2 else 0,
               head_dim=head_dim, softmax_scale=-math.log(W))
    q = torch.zeros((1, 1, 64, head_dim))
    k, v = q.clone(), q.clone()
    q[..., 0] = -1
    k[:, :, 1:, 0] = 1
    v[:, :, 0] = 1
    q, k, v = (x.bfloat16().cuda() for x in (q, k, v))
    out = op.forward(q, k, v)
    torch.cuda.synchronize()
    assert bool((out.float() == OUT).all()), (float(out.float().min()) * 2048, float(out.float().max()) * 2048)
