"""The group kernels' index functions (host build) at the edges of what they
take: one chunk, groups that straddle blocks or end inside one, odd cell
columns, single rows and columns of cells, list tables that fill their 768
rows; and that the checks catch mistakes planted in the expected sets."""
import pytest

import group_emulation as ge
import host_groups as hg
import test_issue_emulation as plans

CASES = [
    # ndim, causal, n or (rows, columns), r, rank, per_level, head_dim
    (1, False, 32, 32, 1, False, 64), (1, True, 32 * 13, 32, 1, False, 64), (1, False, 32 * 37, 32, 4, False, 128),
    (1, True, 32 * 21, 32, 1, True, 32), (1, True, 64 * 5, 64, 2, False, 64), (1, False, 64 * 1024, 64, 6, True, 64),
    (1, False, 192 * 5, 192, 1, False, 128), (1, True, 192 * 7, 192, 2, False, 64), (1, True, 256 * 5, 256, 1, False, 32),
    (1, False, 32 << 16, 32, 4, False, 64),
    (2, False, (24, 40), 8, 1, False, 32), (2, False, (40, 72), 8, 2, False, 128), (2, False, (40, 56), 8, 1, True, 64),
    (2, False, (8, 72), 8, 1, False, 64), (2, False, (72, 8), 8, 1, True, 64), (2, False, (16, 16), 8, 2, True, 64),
    (2, False, (48, 80), 16, 2, False, 64), (2, False, (48, 80), 16, 1, True, 128), (2, False, (8, 32768), 8, 1, True, 64),
    (2, False, (32, 32), 8, 16, False, 64),
]


def _plan(c):
    ndim, causal, size, r, rank, per_level, d = c
    return plans._params(ndim, causal, "bf16", 1, 2, size, r, rank, per_level, head_dim=d)


@pytest.mark.parametrize("case", CASES)
def test_groups_at_their_edges(case):
    P = _plan(case)
    assert hg.attend_kernels(hg.plan_values(P)) & hg.GROUPS
    ge.check_attend(P)
    if P["head_dim"] == 64:
        ge.check_backward(P)


@pytest.mark.parametrize("case", [CASES[1], CASES[6], CASES[11], CASES[12], CASES[16]])
@pytest.mark.parametrize("what", ["tokens", "near", "lists"])
def test_checks_catch_planted_mistakes(case, what, monkeypatch):
    """One token of a block, of its near field or one list row too few."""
    P = _plan(case)
    good = getattr(ge.Geometry, what)

    def bad(self, b):
        x = good(self, b)
        if what != "lists":
            return x[1:]
        for level in x:
            for rows in level:
                if rows:
                    rows.pop()
                    return x
        return x

    monkeypatch.setattr(ge.Geometry, what, bad)
    with pytest.raises(AssertionError):
        ge.check_attend(P)
