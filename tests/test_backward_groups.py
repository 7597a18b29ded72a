"""CPU restatement of the row groups of the bf16 backward (row_groups.hpp):
which tokens every workgroup loads and which of them each wave takes, against
the definition of the near field, for every block size the groups accept."""
import pytest


def row_group(ndim, r, n, nbx, nby, causal, g, wave, keys):
    """row_group<GEOM, KEYS> for 1D, 2D pairs of 8 x 8 cells, halves of 16 x 16 cells."""
    m = dict(lo=0, wlo=0, whi=0, wdiag=-1, x0=0, y0=0, ncx=1, cy=0)
    if ndim == 1:
        f0 = 128 * g
        w0 = f0 + 32 * wave
        l0 = f0 + 96 if f0 + 96 < n else n - 32

        def lo_of(row):
            if keys and causal:
                return row
            b = row // r
            return (b - 1) * r if b > 0 else 0

        def hi_of(row):
            if not keys and causal:
                return row + 32
            return min((row // r + 2) * r, n)
        m["active"] = w0 < n
        m["blk"] = w0 // r if m["active"] else 0
        m["pos0"] = w0 - m["blk"] * r
        lo, hi = lo_of(f0), hi_of(l0)
        m["lo"], m["ntile"] = lo, (hi - lo + 63) // 64
        if m["active"]:
            m["wlo"], m["whi"] = lo_of(w0) - lo, hi_of(w0) - lo
            if causal:
                m["wdiag"] = w0 - lo
    elif r == 8:
        npc = (nby + 1) // 2
        cx, c0, side = g // npc, 2 * (g % npc), wave >> 1
        m["active"] = c0 + side < nby
        m["cy"] = c0 + side
        m["blk"] = cx * nby + m["cy"] if m["active"] else 0
        m["pos0"] = 32 * (wave & 1)
        m["x0"] = max(cx - 1, 0)
        m["ncx"] = min(cx + 1, nbx - 1) - m["x0"] + 1
        m["y0"] = max(c0 - 1, 0)
        m["ntile"] = m["ncx"] * (min(c0 + 2, nby - 1) - m["y0"] + 1)
    else:
        cell = g >> 1
        cx, cy = cell // nby, cell % nby
        m.update(active=True, cy=cy, blk=cell, pos0=128 * (g & 1) + 32 * wave)
        m["x0"] = max(cx - 1, 0)
        m["ncx"] = min(cx + 1, nbx - 1) - m["x0"] + 1
        m["y0"] = max(cy - 1, 0)
        m["ntile"] = 4 * m["ncx"] * (min(cy + 1, nby - 1) - m["y0"] + 1)
    return m


def window_col(r, nby, m, cc):
    if r == 8 and nby % 2 == 0:
        c0 = m["cy"] & ~1
        return c0 + cc if cc < 2 else c0 - 1 if cc == 2 and m["y0"] < c0 else c0 + 2
    return m["y0"] + cc


def tile_run(ndim, r, n, W, m, t, i):
    if ndim == 1:
        tok = m["lo"] + 64 * t + 8 * i
        return tok if tok + 8 <= n else n - 8
    if r == 8:
        col, row = window_col(r, W // 8, m, t // m["ncx"]), t % m["ncx"]
        return ((m["x0"] + row) * 8 + i) * W + col * 8
    c, p0 = t >> 2, (t & 3) * 64 + 8 * i
    col, row = c // m["ncx"], c % m["ncx"]
    return ((m["x0"] + row) * 16 + (p0 >> 4)) * W + (m["y0"] + col) * 16 + (p0 & 15)


def tile_used(ndim, r, nby, m, t, hb):
    if not m["active"]:
        return False
    if ndim == 1:
        return m["wlo"] <= 64 * t + 32 * hb < m["whi"]
    if r == 8:
        return abs(window_col(r, nby, m, t // m["ncx"]) - m["cy"]) <= 1
    return True


def groups(ndim, r, n, nbx, nby):
    return (n + 127) // 128 if ndim == 1 else nbx * ((nby + 1) // 2) if r == 8 else 2 * nbx * nby


def wave_token(ndim, r, W, nby, m, p):
    if ndim == 1:
        return m["blk"] * r + p
    cx, cy = m["blk"] // nby, m["blk"] % nby
    return (cx * r + p // r) * W + cy * r + p % r


SHAPES = [(1, r, r * b, 0, 0, c) for r in (32, 64, 96, 128, 160, 192, 224, 256) for b in (1, 2, 3, 4, 5, 7, 10)
          for c in (False, True)]
SHAPES += [(2, 8, 64 * x * y, x, y, False) for x in (1, 2, 3, 5) for y in (1, 2, 3, 4, 7)]
SHAPES += [(2, 16, 256 * x * y, x, y, False) for x in (1, 2, 4) for y in (1, 2, 3)]


@pytest.mark.parametrize("keys", [False, True])
@pytest.mark.parametrize("ndim,r,n,nbx,nby,causal", SHAPES)
def test_groups_cover_near_window(ndim, r, n, nbx, nby, causal, keys):
    W = nby * r if ndim == 2 else 0
    seen = set()
    for g in range(groups(ndim, r, n, nbx, nby)):
        for wave in range(4):
            m = row_group(ndim, r, n, nbx, nby, causal, g, wave, keys)
            assert m["ntile"] >= 1
            for t in range(m["ntile"]):
                for i in range(8):   # every load stays in the slice
                    assert 0 <= tile_run(ndim, r, n, W, m, t, i) <= n - 8
            if not m["active"]:
                continue
            own = [wave_token(ndim, r, W, nby, m, m["pos0"] + x) for x in range(32)]
            assert not seen & set(own)
            seen |= set(own)
            got = []
            for t in range(m["ntile"]):
                for hb in range(2):
                    if tile_used(ndim, r, nby, m, t, hb):
                        rows = [tile_run(ndim, r, n, W, m, t, 4 * hb + x // 8) + x % 8 for x in range(32)]
                        if causal and 64 * t + 32 * hb == m["wdiag"]:
                            assert rows == own
                        got += rows
            if ndim == 1:
                b = m["blk"]
                want = set(range(max(b - 1, 0) * r, min((b + 2) * r, n)))
                if causal:   # queries at or after the chunk (key pass), keys up to it (query pass)
                    want = {x for x in want if (x >= own[0] if keys else x <= own[-1])}
            else:
                cx, cy = m["blk"] // nby, m["blk"] % nby
                want = {(u * r + p // r) * W + v * r + p % r for u in range(cx - 1, cx + 2) for v in range(cy - 1, cy + 2)
                        if 0 <= u < nbx and 0 <= v < nby for p in range(r * r)}
            assert len(got) == len(set(got)) and set(got) == want
    assert seen == set(range(n))


# ------------------------------------------------ sibling groups' coarse slots
def list1d(b, l, j, M, causal):
    q = b >> (l - 1)
    p = q >> 1
    g = (2 * p - 2 if j == 0 else 2 * p + 1 + j) if q & 1 == 0 else (2 * p + 3 if j == 2 else 2 * p - 2 + j)
    return -1 if g < 0 or g >= M or (causal and g > q - 2) else g


def window_slot(j, ox, oy):
    if j < 6 * ox:
        return j // 6, j % 6
    if j < 6 * ox + 9:
        t = j - 6 * ox
        return ox + t // 3, t % 3 if t % 3 < oy else t % 3 + 3
    t = j - 6 * ox - 9
    return ox + 3 + t // 6, t % 6


def list2d(cx, cy, l, j, Mx, My):
    qx, qy = cx >> (l - 1), cy >> (l - 1)
    au, av = window_slot(j, 1 + (qx & 1), 1 + (qy & 1))
    u, v = 2 * (qx >> 1) - 2 + au, 2 * (qy >> 1) - 2 + av
    return u * My + v if 0 <= u < Mx and 0 <= v < My else -1


def list2d_slot_of(qx, qy, u, v):
    au, av = u - (2 * (qx >> 1) - 2), v - (2 * (qy >> 1) - 2)
    if not (0 <= au < 6 and 0 <= av < 6):
        return -1
    ox, oy = 1 + (qx & 1), 1 + (qy & 1)
    if au < ox:
        return au * 6 + av
    if au < ox + 3:
        return -1 if oy <= av < oy + 3 else 6 * ox + (au - ox) * 3 + (av if av < oy else av - 3)
    return 6 * ox + 9 + (au - ox - 3) * 6 + av


def hierarchy(ndim, nbx, nby, p):
    L, off, sets = 0, 0, []
    while (1 << L) < max(nbx, nby):
        L += 1
    for l in range(1, L):
        s = 1 << (l - 1)
        M, My = -(-nbx // s), 1 if ndim == 1 else -(-nby // s)
        for _ in range(p):
            sets.append((l, M, My, off))
            off += M * My
    return sets, off


def group_slot(ndim, sets, p, nbx, nby, causal, grp, slot):
    """(coarse row, mask of the group's blocks that list it) of a sibling group's slot (bwd_coarse_mfma)."""
    K, KW = (3, 6) if ndim == 1 else (27, 36)
    ngy = (nby + 1) >> 1
    cx0, cy0 = (2 * grp, 0) if ndim == 1 else (2 * (grp // ngy), 2 * (grp % ngy))
    if slot < p * KW:
        l, M, My, off = sets[slot // KW]
        pos = slot % KW
        u, v = (cx0 - 2 + pos, 0) if ndim == 1 else (cx0 - 2 + pos // 6, cy0 - 2 + pos % 6)
        if not (0 <= u < M and 0 <= v < My):
            return -1, 0
        mask = 0
        for i in range(2):
            for j in range(1 if ndim == 1 else 2):
                du, dv = u - cx0 - i, v - cy0 - j
                near = abs(du) <= 1 and (ndim == 1 or abs(dv) <= 1)
                if causal:
                    near = du > -2
                mask |= 0 if near else 1 << (2 * i + j)
        return off + u * My + v, mask
    e = p + (slot - p * KW) // K
    l, M, My, off = sets[e]
    j = (slot - p * KW) % K
    g = list1d(cx0, l, j, M, causal) if ndim == 1 else list2d(cx0, cy0, l, j, M, My)
    return (-1, 0) if g < 0 else (off + g, 15)


def reduce_terms(ndim, sets, p, nbx, nby, causal, crow):
    """(group, slot) partial rows bwd_group_reduce adds for a coarse row."""
    K, KW = (3, 6) if ndim == 1 else (27, 36)
    e = max(x for x in range(len(sets)) if sets[x][3] <= crow)
    l, M, My, off = sets[e]
    g = crow - off
    u, v = (g, 0) if ndim == 1 else (g // My, g % My)
    ngx, ngy = (nbx + 1) >> 1, 1 if ndim == 1 else (nby + 1) >> 1
    out = []
    if l == 1:
        for px in range(max((u >> 1) - 1, 0), min((u >> 1) + 1, ngx - 1) + 1):
            for py in range(max((v >> 1) - 1, 0), min((v >> 1) + 1, ngy - 1) + 1):
                au, av = u - (2 * px - 2), v - (2 * py - 2)
                assert 0 <= au < 6 and (ndim == 1 or 0 <= av < 6)
                out.append((px * ngy + py, e * KW + (au if ndim == 1 else au * 6 + av)))
        return out
    span = 1 << (l - 2)
    for qx in range(u - 3, u + 4):
        for qy in range(v - 3, v + 4) if ndim == 2 else [0]:
            if not (0 <= qx < M and qx * span < ngx and 0 <= qy < My and qy * span < ngy):
                continue
            j = list2d_slot_of(qx, qy, u, v) if ndim == 2 else max(
                [j for j in range(3) if list1d(2 * qx * span, l, j, M, causal) == g], default=-1)
            if j >= 0:
                out += [(px * ngy + py, p * KW + (e - p) * K + j)
                        for px in range(qx * span, min((qx + 1) * span, ngx))
                        for py in range(qy * span, min((qy + 1) * span, ngy))]
    return out


@pytest.mark.parametrize("ndim,nbx,nby,p,causal", [
    (1, 3, 1, 1, False), (1, 4, 1, 1, True), (1, 9, 1, 2, False), (1, 23, 1, 1, True), (1, 32, 1, 3, False),
    (1, 37, 1, 1, False), (2, 3, 3, 1, False), (2, 5, 7, 1, False), (2, 1, 9, 1, False), (2, 9, 1, 2, False),
    (2, 16, 16, 1, False), (2, 4, 13, 3, False), (2, 15, 21, 1, False)])
def test_sibling_groups_hold_every_list(ndim, nbx, nby, p, causal):
    """Every block's interaction list is what its sibling group's slots show
    it, and every coarse row collects exactly the groups that list it."""
    K, KW = (3, 6) if ndim == 1 else (27, 36)
    sets, R = hierarchy(ndim, nbx, nby, p)
    gslot = p * KW + (len(sets) - p) * K
    ngy = 1 if ndim == 1 else (nby + 1) >> 1
    ngrp = ((nbx + 1) >> 1) * ngy
    pairs = set()
    for grp in range(ngrp):
        rows = [group_slot(ndim, sets, p, nbx, nby, causal, grp, s) for s in range(gslot)]
        for i in range(2):
            for j in range(1 if ndim == 1 else 2):
                cx, cy = (2 * grp + i, 0) if ndim == 1 else (2 * (grp // ngy) + i, 2 * (grp % ngy) + j)
                if cx >= nbx or cy >= nby:
                    continue
                got = sorted(r for r, m in rows if (m >> (2 * i + j)) & 1)
                want = sorted(off + g for l, M, My, off in sets for x in range(K)
                              for g in [list1d(cx, l, x, M, causal) if ndim == 1 else list2d(cx, cy, l, x, M, My)]
                              if g >= 0)
                assert got == want
        for s, (r, m) in enumerate(rows):
            assert r < R
            if m:
                pairs.add((grp, s, r))
    terms = set()
    for r in range(R):
        for g, s in reduce_terms(ndim, sets, p, nbx, nby, causal, r):
            assert 0 <= g < ngrp and 0 <= s < gslot
            assert (g, s, r) not in terms
            terms.add((g, s, r))
            # a row it reads was stored for this coarse row, or is all zeros
            row, m = group_slot(ndim, sets, p, nbx, nby, causal, g, s)
            assert row == r or m == 0
    assert pairs <= terms
