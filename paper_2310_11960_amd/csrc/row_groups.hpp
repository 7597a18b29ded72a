// row_groups.hpp -- groups of 128 rows that a workgroup of the bf16 streaming
// kernels (forward and backward) owns, the near windows they walk, and the
// groups' interaction-list rows.
//
// A workgroup of four waves owns a group of 128 rows (queries of the query
// pass, keys of the key pass), 32 consecutive rows of one base block per wave:
//   1D        128 consecutive tokens, whatever the block size (a multiple of
//             32): blocks of 32 and 64 share a workgroup, larger ones split;
//   2D, r = 8 two horizontally adjacent cells (cx, 2c), (cx, 2c + 1), whose
//             3x3 near windows share six cells; the last pair of an odd row
//             has no right cell and its waves only help to load;
//   2D, r = 16 half a cell (eight rows of it).
// The rows of the group's near window are loaded once for all waves; a wave
// takes the 32-row pieces that lie in its own window.  Eight rows of the
// window that start at a multiple of eight are consecutive tokens.
#pragma once

#include "fma_device.hpp"
#include "fma_kernels.hpp"

namespace fma_dev {

namespace {

// 16 bytes (4 bytes) per lane from global memory to LDS byte lds_base + 16 L
// (4 L).  Inline assembly: the compiler does not order later LDS reads
// behind these loads, the loops wait for them explicitly (wait_vm).
__device__ __attribute__((always_inline)) inline void dma16(const void *gptr, uint32_t lds_base)
{
    asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(gptr), "{m0}"(lds_base) : "memory");
}
__device__ __attribute__((always_inline)) inline void dma4(const void *gptr, uint32_t lds_base)
{
    asm volatile("global_load_lds_dword %0, off" : : "v"(gptr), "{m0}"(lds_base) : "memory");
}

// wait until at most N vector-memory operations of this wave are in flight
template <int N>
__device__ __attribute__((always_inline)) inline void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __attribute__((always_inline)) inline uint32_t lds_u32(const void *p)
{
    return __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void *)p)));
}

// Position of workgroup `bid` of `total` when the eight XCDs, which take
// workgroups round-robin, each walk one contiguous range: neighbouring groups,
// which share most of their near window, meet in one XCD's L2.
__host__ __device__ __attribute__((always_inline)) inline unsigned xcd_contiguous(unsigned bid, unsigned total)
{
    const unsigned x = bid & 7, j = bid >> 3, per = total >> 3, rem = total & 7;
    return x * per + (x < rem ? x : rem) + j;
}

// A group of 128 rows: its window, in 32-row pieces, and this wave's part.
struct RowGroup {
    int npiece;           // 32-row pieces of the near window
    int wlo, whi;         // 1D: this wave's part of the window, rows [wlo, whi) (2D: see piece_used)
    int wdiag;            // causal 1D: the window row where the wave's own rows start
    bool active;          // the wave has rows
    int blk;              // the wave's base block (1D) or cell (cx * nby + cy)
    int pos0;             // position of the wave's first row in that block (1D: token, 2D: pixel)
    long long lo;         // 1D: first token of the window
    int x0, y0, ncx, cy;  // 2D: first cell row / column of the window, its cell rows; the wave's cell column
};

// Groups per slice.
template <int GEOM, typename A>
__host__ __device__ inline long long row_groups(const A &a)
{
    if (GEOM == GEOM_1D) return (a.n + 127) / 128;
    if (GEOM == GEOM_2DP) return (long long)a.nbx * ((a.nby + 1) / 2);
    return 2LL * a.nbx * a.nby;
}

// Group g seen by wave `wave`.  KEYS: rows are keys and the window holds the
// queries that may see them (causal: those at or after the key); else rows
// are queries and the window holds their near keys.
template <int GEOM, bool KEYS, typename A>
__host__ __device__ __attribute__((always_inline)) inline RowGroup row_group(const A &a, int g, int wave)
{
    RowGroup m;
    m.lo = 0;
    m.x0 = m.y0 = m.cy = 0;
    m.ncx = 1;
    m.wlo = 0;
    m.whi = 0;
    m.wdiag = -1;
    if constexpr (GEOM == GEOM_1D) {
        const int n = (int)a.n, r = a.r;   // tokens fit 31 bits (the launcher checks)
        const int f0 = 128 * g, w0 = f0 + 32 * wave;
        const int l0 = f0 + 96 < n ? f0 + 96 : n - 32;   // first row of the last active wave
        auto lo_of = [&](int row) {
            if (KEYS && a.causal) return row;
            const int b = row / r;
            return b > 0 ? (b - 1) * r : 0;
        };
        auto hi_of = [&](int row) {
            if (!KEYS && a.causal) return row + 32;
            const int h = (row / r + 2) * r;
            return h < n ? h : n;
        };
        m.active = w0 < n;
        m.blk = m.active ? w0 / r : 0;
        m.pos0 = w0 - m.blk * r;
        const int lo = lo_of(f0), hi = hi_of(l0);
        m.lo = lo;
        m.npiece = (hi - lo) / 32;
        if (m.active) {
            m.wlo = lo_of(w0) - lo;
            m.whi = hi_of(w0) - lo;
            if (a.causal) m.wdiag = w0 - lo;
        }
    } else if constexpr (GEOM == GEOM_2DP) {
        const int npc = (a.nby + 1) >> 1;
        const int cx = g / npc, c0 = 2 * (g - cx * npc), side = wave >> 1;
        m.active = c0 + side < a.nby;
        m.cy = c0 + side;
        m.blk = m.active ? cx * a.nby + m.cy : 0;
        m.pos0 = 32 * (wave & 1);
        m.x0 = cx > 0 ? cx - 1 : 0;
        m.ncx = (cx + 1 < a.nbx ? cx + 1 : cx) - m.x0 + 1;
        m.y0 = c0 > 0 ? c0 - 1 : 0;
        const int y1 = c0 + 2 < a.nby ? c0 + 2 : a.nby - 1;
        m.npiece = 2 * m.ncx * (y1 - m.y0 + 1);
    } else {
        const int cell = g >> 1;
        const int cx = cell / a.nby, cy = cell - cx * a.nby;
        m.active = true;
        m.cy = cy;
        m.blk = cell;
        m.pos0 = 128 * (g & 1) + 32 * wave;
        m.x0 = cx > 0 ? cx - 1 : 0;
        m.ncx = (cx + 1 < a.nbx ? cx + 1 : cx) - m.x0 + 1;
        m.y0 = cy > 0 ? cy - 1 : 0;
        const int y1 = cy + 1 < a.nby ? cy + 1 : cy;
        m.npiece = 8 * m.ncx * (y1 - m.y0 + 1);
    }
    return m;
}

// 2D: cell column of the window's cc-th column.  Pairs of an even row: the two
// columns that both cells see first, then the left cell's, then the right
// cell's, so that both cells start from the same cell; else ascending.
template <int GEOM, typename A>
__host__ __device__ __attribute__((always_inline)) inline int window_col(const A &a, const RowGroup &m, int cc)
{
    if constexpr (GEOM == GEOM_2DP) {
        if (a.nby % 2 == 0) {
            const int c0 = m.cy & ~1, left = m.y0 < c0 ? 1 : 0;
            return cc < 2 ? c0 + cc : cc == 2 && left ? c0 - 1 : c0 + 2;
        }
    }
    return m.y0 + cc;
}

// First token of rows 8 x .. 8 x + 7 of the window (2D: column by column of its
// cells); rows past the window stay in the sequence (1D: repeat its end) or map
// (2D: the caller stops at whole cells).
template <int GEOM, typename A>
__host__ __device__ __attribute__((always_inline)) inline long long window_run(const A &a, const RowGroup &m, int x)
{
    if constexpr (GEOM == GEOM_1D) {
        const long long tok = m.lo + 8 * (long long)x;
        return tok + 8 <= a.n ? tok : a.n - 8;
    } else if constexpr (GEOM == GEOM_2DP) {
        const int t = x >> 3, cc = t / m.ncx, row = t - cc * m.ncx;
        return (long long)((m.x0 + row) * 8 + (x & 7)) * a.side + window_col<GEOM>(a, m, cc) * 8;
    } else {
        const int c = x >> 5, p0 = 8 * (x & 31);
        const int col = c / m.ncx, row = c - col * m.ncx;
        return (long long)((m.x0 + row) * 16 + (p0 >> 4)) * a.side + (m.y0 + col) * 16 + (p0 & 15);
    }
}

// Row `row` of tile t (TR rows) of the attention's near window: 1D consecutive
// tokens, the last of the sequence repeated past its end; 2D pixel p0 + row of
// the tile's cell (whole cells, so that no tile leaves the window).
struct TileCell {
    long long base;   // 2D: first token of the cell
    int p0;
};
template <int GEOM, int TR, typename A>
__host__ __device__ __attribute__((always_inline)) inline TileCell tile_cell(const A &a, const RowGroup &m, int t)
{
    TileCell r = {0, 0};
    if constexpr (GEOM != GEOM_1D) {
        constexpr int lg = GEOM == GEOM_2DP ? 3 : 4;
        const int c = (t * TR) >> (2 * lg), cc = c / m.ncx, row = c - cc * m.ncx, col = window_col<GEOM>(a, m, cc);
        r.p0 = (t * TR) & ((1 << 2 * lg) - 1);
        r.base = (long long)((m.x0 + row) << lg) * a.side + (col << lg);
    }
    return r;
}
template <int GEOM, int TR, typename A>
__host__ __device__ __attribute__((always_inline)) inline long long tile_token(const A &a, const RowGroup &m, const TileCell &c, int t, int row)
{
    if constexpr (GEOM == GEOM_1D) {
        const long long tok = m.lo + (long long)t * TR + row;
        return tok < a.n ? tok : a.n - 1;
    } else {
        constexpr int lg = GEOM == GEOM_2DP ? 3 : 4;
        const int p = c.p0 + row;
        return c.base + (long long)(p >> lg) * a.side + (p & ((1 << lg) - 1));
    }
}

// Whether this wave takes piece p (rows 32 p .. 32 p + 31) of the window.
template <int GEOM, typename A>
__host__ __device__ __attribute__((always_inline)) inline bool piece_used(const A &a, const RowGroup &m, int p)
{
    if (!m.active) return false;
    if constexpr (GEOM == GEOM_1D) {
        return 32 * p >= m.wlo && 32 * p < m.whi;
    } else if constexpr (GEOM == GEOM_2DP) {
        const int d = window_col<GEOM>(a, m, (p >> 1) / m.ncx) - m.cy;
        return d >= -1 && d <= 1;
    } else {
        return true;
    }
}

// Token of position p of the wave's base block
template <int GEOM, typename A>
__host__ __device__ __attribute__((always_inline)) inline long long wave_token(const A &a, const RowGroup &m, int p)
{
    if constexpr (GEOM == GEOM_1D) {
        return (long long)m.blk * a.r + p;
    } else {
        constexpr int lg = GEOM == GEOM_2DP ? 3 : 4;
        const int cx = m.blk / a.nby, cy = m.blk - cx * a.nby;
        return (long long)((cx << lg) + (p >> lg)) * a.side + (cy << lg) + (p & ((1 << lg) - 1));
    }
}

// Coarse-set tables in LDS (indexing the argument block with a computed
// index per lane costs scattered loads or a copy to scratch)
struct SetTab {
    int lvl[kMaxSets], M[kMaxSets], My[kMaxSets], off[kMaxSets], size[kMaxSets], woff[kMaxSets];
};
template <typename A>
__device__ __attribute__((always_inline)) inline void load_sets(SetTab &t, const A &a, int tid)
{
    if (tid < a.lv.nlev && tid < kMaxSets) {
        t.lvl[tid] = a.lv.lvl[tid];
        t.M[tid] = a.lv.M[tid];
        t.My[tid] = a.lv.My[tid];
        t.off[tid] = a.lv.off[tid];
        t.size[tid] = a.lv.size[tid];
        t.woff[tid] = a.lv.woff[tid];
    }
}


// List rows of a query group, in 32-row pieces: 1D every block's own list, one
// after the other; 2D pairs the slots of their sibling group (group_slots:
// level-1 window, shared lists), seen by each cell through a bit mask; 16 x 16
// cells their own list.  PL (per-level normalisation, levels padded to
// slot_group slots): every block's or cell's own list, also for pairs.
constexpr int kGroupRows = 768;   // most list rows (group_lists_fit): 1D 4 blocks of 32 x 192, 2D joint 576, PL pairs 2 x 384

struct GroupLists {
    int nslot;            // slots per list
    int npc;              // pieces per list
    int npiece;           // pieces of the group
    int pc0;              // this wave's first piece (it takes npc)
    int b0, nb;           // 1D: first block of the group, blocks
};

// An empty row of a piece that has others repeats one of them: its weight is
// 0, and what it loads is a row that the queries see anyway, so that a coarse
// row that is not finite reaches no query that does not list it (0 * inf is
// NaN).  Pieces without a row the kernels skip.
struct ListSmem {
    int crow[kGroupRows];             // coarse row of every list row (-1: a piece without rows)
    uint32_t vis[2][kGroupRows / 32]; // rows each cell of a 2D pair sees (else [0])
};

template <int GEOM, bool PL = false, typename A>
__host__ __device__ __attribute__((always_inline)) inline GroupLists group_lists(const A &a, const RowGroup &m, int grp, int wave = 0)
{
    GroupLists l;
    l.b0 = GEOM == GEOM_1D ? 128 * grp / a.r : 0;
    l.nb = GEOM == GEOM_1D ? (128 * grp + 96 < a.n ? 128 * grp + 96 : (int)a.n - 32) / a.r - l.b0 + 1
                            : GEOM == GEOM_2DP && PL ? 2 : 1;
    l.nslot = a.lv.nlev == 0 ? 0 : GEOM == GEOM_2DP && !PL ? group_slots(1, a.rank, a.lv.nlev) : a.nslot;
    l.npc = (l.nslot + 31) / 32;
    l.npiece = l.nb * l.npc;
    l.pc0 = GEOM == GEOM_1D ? (m.blk - l.b0) * l.npc : GEOM == GEOM_2DP && PL ? (wave >> 1) * l.npc : 0;
    return l;
}

// Coarse row of list row e of a group (-1: empty), and which of a 2D pair's
// cells see it (else bit 0).
template <int GEOM, bool PL = false, typename A, typename T>
__host__ __device__ __attribute__((always_inline)) inline int list_row(const A &a, const RowGroup &m, const GroupLists &l, int grp, const T &st, int e, int &mask)
{
    constexpr int K = GEOM == GEOM_1D ? kSlots1D : kSlots2D;
    int row = -1;
    mask = 0;
    if constexpr (GEOM == GEOM_1D || PL) {
        const int bl = e / (32 * l.npc), sl = e - bl * 32 * l.npc;
        int set = sl / K, j = sl - set * K;
        bool on = bl < l.nb && sl < l.nslot;
        if constexpr (PL) {
            const int lev = sl / a.slot_group, rem = sl - lev * a.slot_group, basis = rem / K;
            set = lev * a.rank + basis;
            j = rem - basis * K;
            on = on && basis < a.rank;
        }
        if (on) {
            int g;
            if constexpr (GEOM == GEOM_1D) {
                g = list1d_entry(l.b0 + bl, st.lvl[set], j, st.M[set], a.causal);
            } else {
                const int npr = (a.nby + 1) >> 1;
                const int cx = GEOM == GEOM_2DP ? grp / npr : m.blk / a.nby;
                const int cy = GEOM == GEOM_2DP ? 2 * (grp - cx * npr) + bl : m.blk - (m.blk / a.nby) * a.nby;
                g = list2d_entry(cx, cy, st.lvl[set], j, st.M[set], st.My[set]);
            }
            if (g >= 0) {
                row = st.off[set] + g;
                mask = 1;
            }
        }
    } else {
        const int cx = GEOM == GEOM_2DP ? grp / ((a.nby + 1) >> 1) : m.blk / a.nby;
        const int cy = GEOM == GEOM_2DP ? 2 * (grp - cx * ((a.nby + 1) >> 1)) : m.blk - (m.blk / a.nby) * a.nby;
        if (e < l.nslot) {
            const int nw = GEOM == GEOM_2DP ? a.rank * group_window(1) : 0;
            if (e < nw) {
                const int set = e / 36, pos = e - set * 36;
                const int u = 2 * (cx >> 1) - 2 + pos / 6, v = 2 * (cy >> 1) - 2 + pos % 6;
                if (u >= 0 && u < st.M[set] && v >= 0 && v < st.My[set]) {
                    row = st.off[set] + u * st.My[set] + v;
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int du = u - cx, dv = v - cy - c;
                        mask |= (du < -1 || du > 1 || dv < -1 || dv > 1) ? 1 << c : 0;
                    }
                }
            } else {
                const int set = (GEOM == GEOM_2DP ? a.rank : 0) + (e - nw) / K, j = (e - nw) % K;
                const int g = list2d_entry(cx, cy, st.lvl[set], j, st.M[set], st.My[set]);
                if (g >= 0) {
                    row = st.off[set] + g;
                    mask = 3;
                }
            }
        }
    }
    return row;
}

// Rows of a group's list table: its pieces, in pairs.
__host__ __device__ __attribute__((always_inline)) inline int list_table_rows(const GroupLists &l) { return (l.npiece + 1) / 2 * 64; }

// Fill the group's list table by four waves.
template <int GEOM, bool PL = false, typename A>
__device__ __attribute__((always_inline)) inline void build_lists(const A &a, const RowGroup &m, const GroupLists &l, int grp,
                                                                  const SetTab &st, int wave, int lane, ListSmem &ls)
{
    const int rows = list_table_rows(l);
    for (int e0 = 64 * wave; e0 < rows; e0 += 256) {
        const int e = e0 + lane;
        int mask;
        const int row = list_row<GEOM, PL>(a, m, l, grp, st, e, mask);
        const uint32_t on32 = (uint32_t)(__builtin_amdgcn_ballot_w64(row >= 0) >> (lane & 32));
        const int sub = __shfl(row, (lane & 32) + (on32 ? __builtin_ctz(on32) : 0));
        ls.crow[e] = row < 0 ? sub : row;
#pragma unroll
        for (int c = 0; c < (GEOM == GEOM_2DP ? 2 : 1); ++c) {
            const unsigned long long b = __builtin_amdgcn_ballot_w64((mask >> c) & 1);
            if (lane == 0) {
                ls.vis[c][e0 / 32] = (uint32_t)b;
                ls.vis[c][e0 / 32 + 1] = (uint32_t)(b >> 32);
            }
        }
    }
}

// A sibling group of base blocks (group_slots): 1D blocks 2 grp, 2 grp + 1; 2D
// the 2 x 2 cells of a parent square, fewer at the end of the map.
struct SiblingGroup {
    int cx0, cy0;   // its first block / cell
    int ncx, ncy;   // blocks per axis
    int cpb;        // 32-row chunks per block
    int lgr;        // log2 of the cell side
};
template <bool TWO_D, typename A>
__host__ __device__ __attribute__((always_inline)) inline SiblingGroup sibling_group(const A &a, int grp)
{
    SiblingGroup s;
    s.cx0 = 2 * grp;
    s.cy0 = 0;
    s.ncy = 1;
    s.lgr = 31 - __builtin_clz(a.r);
    if constexpr (TWO_D) {
        const int ngy = (a.nby + 1) >> 1;
        s.cx0 = 2 * (grp / ngy);
        s.cy0 = 2 * (grp - (grp / ngy) * ngy);
        s.ncy = a.nby - s.cy0 < 2 ? 1 : 2;
        s.cpb = a.r * a.r / 32;
    } else {
        s.cpb = a.r / 32;
    }
    s.ncx = a.nbx - s.cx0 < 2 ? 1 : 2;
    return s;
}
// Block (i, j) of the group's chunk c and the chunk's position p in it
__host__ __device__ __attribute__((always_inline)) inline void sibling_block(const SiblingGroup &s, int c, int &i, int &j, int &p)
{
    const int b = c / s.cpb;
    i = b / s.ncy;
    j = b - i * s.ncy;
    p = 32 * (c - b * s.cpb);
}
// First of the eight consecutive tokens of rows 8 i8 .. of chunk c
template <bool TWO_D, typename A>
__host__ __device__ __attribute__((always_inline)) inline long long sibling_run(const A &a, const SiblingGroup &s, int c, int i8)
{
    int i, j, p;
    sibling_block(s, c, i, j, p);
    p += 8 * i8;
    if constexpr (TWO_D)
        return (long long)(((s.cx0 + i) << s.lgr) + (p >> s.lgr)) * a.side + ((s.cy0 + j) << s.lgr) + (p & (a.r - 1));
    else
        return (long long)(s.cx0 + i) * a.r + p;
}
// Coarse row of a slot of the group (0 where it has none) and the blocks (bit
// 2 i + j) that list it
template <bool TWO_D, typename A>
__host__ __device__ __attribute__((always_inline)) inline int sibling_slot(const A &a, const SiblingGroup &s, int gslot, int slot, int &mask)
{
    constexpr int K = TWO_D ? kSlots2D : kSlots1D;
    mask = 0;
    if (slot >= gslot) return 0;
    const int nw = a.rank * group_window(TWO_D);
    if (slot < nw) {
        const int set = slot / group_window(TWO_D), pos = slot - set * group_window(TWO_D);
        const int u = s.cx0 - 2 + (TWO_D ? pos / 6 : pos), v = TWO_D ? s.cy0 - 2 + pos % 6 : 0;
        if (u < 0 || u >= a.lv.M[set] || (TWO_D && (v < 0 || v >= a.lv.My[set]))) return 0;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < (TWO_D ? 2 : 1); ++j) {
                const int du = u - s.cx0 - i, dv = v - s.cy0 - j;
                bool near = du >= -1 && du <= 1 && (!TWO_D || (dv >= -1 && dv <= 1));
                if (!TWO_D && a.causal) near = du > -2;
                mask |= near ? 0 : 1 << (2 * i + j);
            }
        return a.lv.off[set] + (TWO_D ? u * a.lv.My[set] + v : u);
    }
    const int set = a.rank + (slot - nw) / K, j = (slot - nw) % K;
    int g;
    if constexpr (TWO_D)
        g = list2d_entry(s.cx0, s.cy0, a.lv.lvl[set], j, a.lv.M[set], a.lv.My[set]);
    else
        g = list1d_entry(s.cx0, a.lv.lvl[set], j, a.lv.M[set], a.causal);
    if (g < 0) return 0;
    mask = 15;
    return a.lv.off[set] + g;
}

// Whether a group's list table fits (host).
template <int GEOM, typename A>
inline bool group_lists_fit(const A &a)
{
    if (a.lv.nlev == 0) return true;
    const bool own = GEOM == GEOM_2DP && a.norm_level;   // a pair's two own lists
    const int nslot = GEOM == GEOM_2DP && !own ? group_slots(1, a.rank, a.lv.nlev) : a.nslot;
    const int lists = GEOM != GEOM_1D ? (own ? 2 : 1) : a.r < 128 ? 128 / a.r : 2;   // lists a group can hold
    return (lists * ((nslot + 31) / 32) + 1) / 2 * 64 <= kGroupRows;
}

}  // namespace

}  // namespace fma_dev
