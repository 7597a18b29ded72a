"""Which kernel runs a bf16 plan's attention (attend_route.hpp), on the CPU:
every plan that fma_plan accepts has one, and calls whose kernel depends on
how they fill the device take the one that measured faster."""
import pytest
import torch

import host_groups as hg
import paper_2310_11960_amd as F


def _plan(**kw):
    """The plan's values, or None where fma_plan refuses it."""
    try:
        op = F.FMA(**{**dict(batch=1, heads=2, dtype=torch.bfloat16), **kw})
    except F.FmaError as e:
        assert e.status in (F.FMA_ERR_UNSUPPORTED, F.FMA_ERR_SHAPE)
        return None
    return hg.plan_values(F.fma_plan_params(op.handle))


def _expected(kw):
    """The kernels a plan may take, from its description alone."""
    d, r, two_d = kw["head_dim"], kw["block"], kw["ndim"] == 2
    return hg.STAGED if d != 64 or r < (8 if two_d else 64) else 0


@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("linear", [False, True])
def test_every_sequence_plan_has_a_kernel(head_dim, linear):
    seen = 0
    for r in (16, 32, 64, 128, 192, 256):
        for nb in (1, 2, 3, 5, 16, 1000, 1 << 16):
            for rank in (1, 2, 3, 5, 6, 10, 16, 64):
                for causal in (False, True):
                    for norm in (F.FMA_NORM_JOINT, F.FMA_NORM_PER_LEVEL):
                        kw = dict(ndim=1, seq_len=r * nb, block=r, causal=causal, head_dim=head_dim, rank=rank, norm=norm,
                                  linear=linear)
                        v = _plan(**kw)
                        if v is None:
                            continue
                        seen += 1
                        k = hg.attend_kernels(v)
                        assert k != 0, kw
                        if k & hg.STAGED:
                            assert k == hg.STAGED and _expected(kw) == hg.STAGED
                        if k & hg.STREAM:   # whole blocks of 2, 4, 6 or 8 waves at d = 64
                            assert head_dim == 64 and r >= (64 if linear else 128)
                        assert not k & hg.PAIRS
    assert seen > 40


@pytest.mark.parametrize("head_dim", [32, 64, 128])
@pytest.mark.parametrize("linear", [False, True])
def test_every_map_plan_has_a_kernel(head_dim, linear):
    seen = 0
    for r in (4, 8, 16):
        for cells in ((1, 1), (1, 2), (2, 2), (2, 1), (1, 3), (3, 5), (5, 8), (16, 16), (1, 4096), (2, 8192), (1, 16384)):
            for rank in (1, 2, 3, 4, 8, 16):
                for norm in (F.FMA_NORM_JOINT, F.FMA_NORM_PER_LEVEL):
                    kw = dict(ndim=2, seq_len=r * r * cells[0] * cells[1], side=r * cells[1], block=r, head_dim=head_dim,
                              rank=rank, norm=norm, linear=linear)
                    v = _plan(**kw)
                    if v is None:
                        continue
                    seen += 1
                    k = hg.attend_kernels(v)
                    assert k in (hg.STAGED, hg.GROUPS, hg.STREAM, hg.PAIRS), kw
                    if k == hg.STAGED:
                        assert _expected(kw) == hg.STAGED
                    if k in (hg.STREAM, hg.PAIRS):
                        assert linear or norm == F.FMA_NORM_PER_LEVEL
    assert seen > 20


# block, causal, slices, blocks per slice, us in groups, us in the stream (256 CUs, d = 64)
MEASURED = [
    (128, False, 8, 32, 12.4, 13.0), (128, False, 128, 4, 15.9, 16.1), (128, False, 64, 10, 19.9, 19.5),
    (128, False, 1, 600, 19.6, 19.2), (128, False, 64, 16, 26.6, 26.0),
    (256, False, 8, 16, 19.8, 20.9), (256, False, 16, 9, 22.5, 20.9), (256, False, 32, 8, 24.6, 21.8),
    (256, False, 17, 9, 23.7, 32.4), (256, False, 32, 9, 28.9, 31.2), (256, False, 64, 6, 29.8, 31.7),
    (256, False, 32, 16, 39.5, 34.8), (256, False, 64, 16, 71.1, 63.9), (256, False, 128, 12, 101.9, 91.3),
    (256, True, 8, 16, 15.0, 17.3), (256, True, 32, 8, 18.6, 18.1), (256, True, 64, 5, 23.1, 24.5),
    (256, True, 32, 16, 29.0, 26.5), (256, True, 64, 16, 49.8, 48.5),
    (192, False, 8, 32, 22.9, 19.4), (192, False, 8, 8, 19.1, 18.7), (192, False, 64, 12, 44.4, 41.0),
    (192, False, 128, 7, 46.2, 58.2), (192, False, 128, 12, 69.6, 84.6),
]


@pytest.mark.parametrize("r,causal,slices,blocks,groups_us,stream_us", MEASURED)
def test_device_filling_rule_takes_the_faster_kernel(r, causal, slices, blocks, groups_us, stream_us):
    v = _plan(ndim=1, heads=slices, batch=1, seq_len=r * blocks, block=r, causal=causal)
    assert hg.attend_kernels(v) == hg.GROUPS | hg.STREAM
    assert hg.groups_win(v) == (groups_us < stream_us)
