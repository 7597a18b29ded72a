"""Empty interaction-list slots add nothing, whatever the coarse rows hold: a
causal query whose list is empty gives the same result, bit for bit, when the
values of later tokens that it cannot see are not finite.  The first 64
queries of a block of 128 share no 64-key tile with the tokens from 64 on."""
import pytest
import torch

import paper_2310_11960_amd as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,r", [(128, 128), (32, 256), (64, 128), (128, 192)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_unseen_values_do_not_leak(head_dim, r, bad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 8 * r
    op = F.FMA(ndim=1, batch=1, heads=2, seq_len=n, block=r, causal=True, dtype=torch.bfloat16, head_dim=head_dim)
    g = torch.Generator().manual_seed(r + head_dim)
    q, k, v = (torch.randn((1, 2, n, head_dim), generator=g).bfloat16().cuda() for _ in range(3))
    wk, wv = ((torch.randn((2, op.weights_len), generator=g) / r ** 0.5).cuda() for _ in range(2))
    want = op.forward(q, k, v, wk, wv)
    v[:, :, r - 1] = bad
    got = op.forward(q, k, v, wk, wv)
    torch.cuda.synchronize()
    assert bool((got[:, :, :64] == want[:, :, :64]).all())
