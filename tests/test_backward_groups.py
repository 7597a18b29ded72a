"""CPU restatement of the row groups of the bf16 backward (bwd_tiles.hpp):
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


def tile_run(ndim, r, n, W, m, t, i):
    if ndim == 1:
        tok = m["lo"] + 64 * t + 8 * i
        return tok if tok + 8 <= n else n - 8
    if r == 8:
        col, row = t // m["ncx"], t % m["ncx"]
        return ((m["x0"] + row) * 8 + i) * W + (m["y0"] + col) * 8
    c, p0 = t >> 2, (t & 3) * 64 + 8 * i
    col, row = c // m["ncx"], c % m["ncx"]
    return ((m["x0"] + row) * 16 + (p0 >> 4)) * W + (m["y0"] + col) * 16 + (p0 & 15)


def tile_used(ndim, r, m, t, hb):
    if not m["active"]:
        return False
    if ndim == 1:
        return m["wlo"] <= 64 * t + 32 * hb < m["whi"]
    if r == 8:
        return abs(m["y0"] + t // m["ncx"] - m["cy"]) <= 1
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
                    if tile_used(ndim, r, m, t, hb):
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
