"""Checks of the row groups that the bf16 group kernels walk (row_groups.hpp,
built for the host by host_groups), for a plan as fma_plan_params gives it:
every load stays in its slice, every wave takes its block's near field once,
and every list table holds exactly the block's interaction lists, rows of
their own sets, in at most the table's size.

The near field and the lists are written out from their definitions here;
group counts and coarse-row offsets come from the block counts, not from the
plan's tables.  Large plans are checked on a sample of groups (the first and
last ones and some between)."""
import numpy as np

import host_groups as hg

GROUP_ROWS = 768   # kGroupRows


def _axis(nb, l, b, causal=False):
    """Level-l groups of one axis next to block b's parent: (group, near)."""
    M, q = (nb + (1 << (l - 1)) - 1) >> (l - 1), b >> (l - 1)
    out = [(g, abs(g - q) <= 1) for g in range(2 * (q >> 1) - 2, 2 * (q >> 1) + 4) if 0 <= g < M]
    return M, q, out


class Geometry:
    def __init__(self, P):
        self.P, self.r, self.n = P, P["block"], P["n"]
        self.two_d, self.causal, self.rank = P["ndim"] == 2, bool(P["causal"]), P["rank"]
        if self.two_d:
            assert P["nbx"] * self.r == P["height"] and P["nby"] * self.r == P["side"] and P["height"] * P["side"] == self.n
            self.nbx, self.nby = P["nbx"], P["nby"]
        else:
            assert P["nbx"] * self.r == self.n
            self.nbx, self.nby = P["nbx"], 1
        levels = max(self.nbx, self.nby)
        self.nlev = max((levels - 1).bit_length() - 1, 0)
        assert P["nsets"] == self.nlev * self.rank
        off = 0
        self.off = []
        for l in range(1, self.nlev + 1):
            s = 1 << (l - 1)
            count = -(-self.nbx // s) * (-(-self.nby // s) if self.two_d else 1)
            for b in range(self.rank):
                e = P["sets"][(l - 1) * self.rank + b]
                assert e["lvl"] == l and e["size"] == self.r * s and e["off"] == off, ("set table", l, b)
                self.off.append(off)
                off += count
        assert off == P["R"], "coarse rows"

    def tokens(self, b):
        r = self.r
        if not self.two_d:
            return np.arange(b * r, (b + 1) * r)
        cx, cy = b // self.nby, b % self.nby
        return ((cx * r + np.arange(r))[:, None] * self.P["side"] + cy * r + np.arange(r)[None, :]).reshape(-1)

    def near(self, b):
        """Tokens of the block's near field, unordered (causal: blocks b - 1, b)."""
        if not self.two_d:
            return np.concatenate([self.tokens(x) for x in range(b - 1, b + 1 if self.causal else b + 2)
                                   if 0 <= x < self.nbx])
        cx, cy = b // self.nby, b % self.nby
        return np.concatenate([self.tokens(u * self.nby + v) for u in range(cx - 1, cx + 2) for v in range(cy - 1, cy + 2)
                               if 0 <= u < self.nbx and 0 <= v < self.nby])

    def lists(self, b):
        """Coarse rows that block b lists, level by level (all bases of a level)."""
        out = []
        for l in range(1, self.nlev + 1):
            if self.two_d:
                _, _, us = _axis(self.nbx, l, b // self.nby)
                My, _, vs = _axis(self.nby, l, b % self.nby)
                gs = [u * My + v for u, nu in us for v, nv in vs if not (nu and nv)]
            else:
                _, q, us = _axis(self.nbx, l, b)
                gs = [g for g, near in us if not near and (not self.causal or g <= q - 2)]
            out.append([[self.off[(l - 1) * self.rank + p] + g for g in gs] for p in range(self.rank)])
        return out


def _sample(total):
    return sorted(set(range(min(total, 12))) | set(range(max(total - 12, 0), total)) | set(range(0, total, max(total // 24, 1))))


def check_near(P, kinds):
    geo, v = Geometry(P), hg.plan_values(P)
    total = hg.group_count(v)
    for kind in kinds:
        keys = kind == hg.KEY
        owned, sample = set(), _sample(total)
        for g in sample:
            for wave in range(4):
                m = hg.group_walk(v, kind, g, wave)
                assert 0 <= m["lo"] and m["hi"] < geo.n, ("load outside the slice", kind, g, wave)
                if not m["active"]:
                    assert len(m["rows"]) == 0
                    continue
                own = m["own"]
                assert set(own) <= set(geo.tokens(m["blk"])) and len(set(own)) == 32
                assert not owned & set(own)
                owned |= set(own)
                want = geo.near(m["blk"])
                if geo.causal:
                    if keys:   # queries from the wave's first key on, of this block and the next
                        hi = min((m["blk"] + 2) * geo.r, geo.n)
                        want = np.arange(own[0], hi)
                    else:      # keys up to the wave's last query
                        want = want[want <= own[-1]]
                    assert m["diag"] >= 0 and (m["rows"][m["diag"]:m["diag"] + 32] == own).all(), "diagonal piece"
                got = np.sort(m["rows"])
                assert len(got) == len(want) and (got == np.sort(want)).all(), ("near field", kind, g, wave)
        if len(sample) == total:
            assert owned == set(range(geo.n)), "rows without a wave"


def check_lists(P, per_level=None):
    geo, v = Geometry(P), hg.plan_values(P)
    pl = bool(P["norm_level"]) if per_level is None else per_level
    if geo.nlev == 0:
        return
    for g in _sample(hg.group_count(v)):
        for wave in range(4):
            m = hg.group_walk(v, hg.ATTEND, g, wave)
            t = hg.group_lists(v, pl, g, wave)
            assert 32 * t["npiece"] <= t["rows"] <= GROUP_ROWS, "list table size"
            assert ((t["crow"] >= -1) & (t["crow"] < P["R"])).all()
            if not m["active"]:
                continue
            assert t["blk"] == m["blk"] and 0 <= t["pc0"] and t["pc0"] + t["npc"] <= t["npiece"]
            lo = 32 * t["pc0"]
            crow, seen = t["crow"][lo:lo + 32 * t["npc"]], t["seen"][lo:lo + 32 * t["npc"]]
            assert (crow[seen] >= 0).all()
            want = geo.lists(m["blk"])
            if pl:   # every level in its own aligned slots
                sg = P["slot_group"]
                assert sg <= 32 and 32 % sg == 0
                for l, rows in enumerate(want):
                    got = crow[l * sg:(l + 1) * sg][seen[l * sg:(l + 1) * sg]]
                    assert sorted(got) == sorted(sum(rows, [])), ("level", l, g, wave)
                assert not seen[geo.nlev * sg:].any()
            else:
                assert sorted(crow[seen]) == sorted(sum(sum(want, []), [])), ("list", g, wave)
            if not geo.two_d or pl:
                # a row that the wave does not see is empty
                assert (crow[~seen] == -1).all()
            else:
                # a merged row that the cell does not list is one of its near squares
                hidden = set(crow[~seen]) - {-1}
                near = {geo.off[p] + u * geo.nby + w for p in range(geo.rank)
                        for u, a in _axis(geo.nbx, 1, m["blk"] // geo.nby)[2] for w, b in _axis(geo.nby, 1, m["blk"] % geo.nby)[2]
                        if a and b}
                assert hidden <= near, ("hidden rows", g, wave)


def check_siblings(P):
    """bwd_coarse_mfma: a group's chunks are its blocks' tokens, each once, and
    its slots show every block exactly its own lists."""
    geo, v = Geometry(P), hg.plan_values(P)
    if geo.nlev == 0:
        return
    ngy = (geo.nby + 1) // 2
    total = (geo.nbx + 1) // 2 * ngy
    for grp in _sample(total):
        s = hg.sibling_group(v, grp)
        assert ((s["tokens"] >= 0) & (s["tokens"] < geo.n)).all()
        assert ((s["rows"] >= 0) & (s["rows"] < P["R"])).all()
        blocks = {}
        for (i, j), tok in zip(s["blocks"], s["tokens"]):
            blocks.setdefault((int(i), int(j)), []).append(tok)
        want = {(i, j) for i in range(2) for j in range(2 if geo.two_d else 1)
                if s["cx0"] + i < geo.nbx and s["cy0"] + j < geo.nby}
        assert set(blocks) == want
        for (i, j), tok in blocks.items():
            b = (s["cx0"] + i) * geo.nby + s["cy0"] + j if geo.two_d else s["cx0"] + i
            assert (np.concatenate(tok) == geo.tokens(b)).all(), ("chunk tokens", grp, i, j)
            got = s["rows"][((s["masks"] >> (2 * i + j)) & 1) == 1]
            assert sorted(got) == sorted(sum(sum(geo.lists(b), []), [])), ("sibling lists", grp, i, j)


def check_attend(P):
    """The group kernel's forward of a plan."""
    check_near(P, [hg.ATTEND_128 if P["head_dim"] == 128 else hg.ATTEND])
    check_lists(P)
    return hg.group_count(hg.plan_values(P)) * P["nslice"]


def check_backward(P):
    """The streamed backward passes (bf16, d = 64, whole 32-row chunks)."""
    check_near(P, [hg.QUERY, hg.KEY])
    if not P["norm_level"] and not P["linear"]:
        check_lists(P, per_level=False)
        check_siblings(P)
