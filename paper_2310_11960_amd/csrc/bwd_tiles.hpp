// bwd_tiles.hpp -- what the bf16 matrix-core backward kernels share: 16-byte
// direct-to-LDS loads, the 128-row groups a workgroup owns and the windows of
// 64-row tiles they walk.
//
// A workgroup of four waves owns a group of 128 rows (queries of the query
// pass, keys of the key pass), 32 consecutive rows of one base block per wave:
//   1D        128 consecutive tokens, whatever the block size (a multiple of
//             32): blocks of 32 and 64 share a workgroup, larger ones split;
//   2D, r = 8 two horizontally adjacent cells (cx, 2c), (cx, 2c + 1), whose
//             3x3 near windows share six cells; the last pair of an odd row
//             has no right cell and its waves only help to load;
//   2D, r = 16 half a cell (eight rows of it).
// The tiles of the group's near window are loaded once for all waves; a wave
// takes the 32-row half tiles that lie in its own window.  Every 8-row piece
// of a tile is eight consecutive tokens, so a load's address is a uniform base
// plus the lane's offset.
#pragma once

#include "bwd_device.hpp"

namespace fma_dev {

namespace {

constexpr int ROWB = 128;          // bytes of a bf16 row of 64 channels
constexpr int TILEE = KT * 64;     // elements of one tile

// 16 bytes (4 bytes) per lane from global memory to LDS byte lds_base + 16 L
// (4 L).  Inline assembly: the compiler does not order later LDS reads
// behind these loads, the loops wait for them explicitly (wait_vm).
__device__ inline void dma16(const void *gptr, uint32_t lds_base)
{
    asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(gptr), "{m0}"(lds_base) : "memory");
}
__device__ inline void dma4(const void *gptr, uint32_t lds_base)
{
    asm volatile("global_load_lds_dword %0, off" : : "v"(gptr), "{m0}"(lds_base) : "memory");
}

// wait until at most N vector-memory operations of this wave are in flight
template <int N>
__device__ inline void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ inline uint32_t lds_u32(const void *p)
{
    return __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void *)p)));
}

// Position of workgroup `bid` of `total` when the eight XCDs, which take
// workgroups round-robin, each walk one contiguous range: neighbouring groups,
// which share most of their near window, meet in one XCD's L2.
__device__ inline unsigned xcd_contiguous(unsigned bid, unsigned total)
{
    const unsigned x = bid & 7, j = bid >> 3, per = total >> 3, rem = total & 7;
    return x * per + (x < rem ? x : rem) + j;
}

// A group of 128 rows: its window of tiles and this wave's part of both.
struct RowGroup {
    int ntile;            // 64-row tiles of the near window
    int wlo, whi;         // this wave's window: rows [wlo, whi) of it (2D: see tile_used)
    int wdiag;            // causal 1D: the window row where the wave's own rows start
    bool active;          // the wave has rows
    int blk;              // the wave's base block (1D) or cell (cx * nby + cy)
    int pos0;             // position of the wave's first row in that block (1D: token, 2D: pixel)
    long long lo;         // 1D: first token of the window
    int x0, y0, ncx, cy;  // 2D: first cell row / column of the window, its cell rows; the wave's cell column
};

// Groups per slice.
template <int GEOM>
__host__ __device__ inline long long row_groups(const BwdArgs &a)
{
    if (GEOM == GEOM_1D) return (a.n + 127) / 128;
    if (GEOM == GEOM_2DP) return (long long)a.nbx * ((a.nby + 1) / 2);
    return 2LL * a.nbx * a.nby;
}

// Group g seen by wave `wave`.  KEYS: rows are keys and the window holds the
// queries that may see them (causal: those at or after the key); else rows
// are queries and the window holds their near keys.
template <int GEOM, bool KEYS>
__device__ inline RowGroup row_group(const BwdArgs &a, int g, int wave)
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
        m.ntile = (hi - lo + KT - 1) / KT;
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
        m.ntile = m.ncx * (y1 - m.y0 + 1);
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
        m.ntile = 4 * m.ncx * (y1 - m.y0 + 1);
    }
    return m;
}

// First token of rows 8 i .. 8 i + 7 of window tile t (2D: column by column
// of the window's cells).  Rows past a 1D sequence's end repeat its last ones.
template <int GEOM>
__device__ inline long long tile_run(const BwdArgs &a, const RowGroup &m, int t, int i)
{
    if constexpr (GEOM == GEOM_1D) {
        const long long tok = m.lo + (long long)t * KT + 8 * i;
        return tok + 8 <= a.n ? tok : a.n - 8;
    } else if constexpr (GEOM == GEOM_2DP) {
        const int col = t / m.ncx, row = t - col * m.ncx;
        return (long long)((m.x0 + row) * 8 + i) * a.side + (m.y0 + col) * 8;
    } else {
        const int c = t >> 2, p0 = (t & 3) * KT + 8 * i;
        const int col = c / m.ncx, row = c - col * m.ncx;
        return (long long)((m.x0 + row) * 16 + (p0 >> 4)) * a.side + (m.y0 + col) * 16 + (p0 & 15);
    }
}

// Whether this wave takes half hb (32 rows) of window tile t.
template <int GEOM>
__device__ inline bool tile_used(const RowGroup &m, int t, int hb)
{
    if (!m.active) return false;
    if constexpr (GEOM == GEOM_1D) {
        const int s0 = t * KT + 32 * hb;
        return s0 >= m.wlo && s0 < m.whi;
    } else if constexpr (GEOM == GEOM_2DP) {
        const int d = m.y0 + t / m.ncx - m.cy;
        return d >= -1 && d <= 1;
    } else {
        return true;
    }
}

// Token of position p of the wave's base block
template <int GEOM>
__device__ inline long long wave_token(const BwdArgs &a, const RowGroup &m, int p)
{
    if constexpr (GEOM == GEOM_1D) {
        return (long long)m.blk * a.r + p;
    } else {
        constexpr int lg = GEOM == GEOM_2DP ? 3 : 4;
        const int cx = m.blk / a.nby, cy = m.blk - cx * a.nby;
        return (long long)((cx << lg) + (p >> lg)) * a.side + (cy << lg) + (p & ((1 << lg) - 1));
    }
}

// Byte offset of this lane's 16 bytes inside rows 8 i .. 8 i + 7 (odd = i & 1)
// so that a linear direct-to-LDS load leaves chunk c of row r at position
// c ^ swz(r).
__device__ inline int dma_lane_off(int lane, int odd)
{
    const int lrow = lane >> 3;
    return lrow * ROWB + 16 * ((lane & 7) ^ swz(lrow + 8 * odd));
}

// Two 16-row halves of an accumulator as bf16 B operands
__device__ inline void pack_b(const f32x16 &w, bf16x8 (&pb)[2])
{
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[hf][e] = static_cast<__bf16>(w[8 * hf + e]);
}

// Byte offsets (from a swizzled tile's row 0) of this lane's transposing reads
// of rows 0 .. 15: [half of the channels][rows 0..7 / 8..15]; see
// contract_rows_tr.
struct TrOff {
    int o[2][2];
};
__device__ inline TrOff tr_offsets(int lane)
{
    TrOff t;
    const int gq = lane >> 4, s4 = lane & 15, j = s4 >> 2, q = s4 & 3;
    const int row = 4 * (gq >> 1) + j;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
        const int chunk = 4 * db + 2 * (gq & 1) + (q >> 1);
        t.o[db][0] = sw_off(row, chunk) + 4 * (q & 1);
        t.o[db][1] = sw_off(row + 8, chunk) + 4 * (q & 1);
    }
    return t;
}

// out_db[ch][n] += sum over rows r = rowbase .. rowbase + 31 of
// tile[r][ch] w[r][n], w as packed B operands
__device__ inline void contract_tr(const __bf16 *tile, const TrOff &to, const bf16x8 (&pb)[2], f32x16 &out0, f32x16 &out1)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const __bf16 *t16 = tile + 16 * hf * kHeadDim;
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            const s16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + to.o[db][0]));
            const s16x4 r2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + to.o[db][1]));
            const s16x8 av = {r1[0], r1[1], r1[2], r1[3], r2[0], r2[1], r2[2], r2[3]};
            const bf16x8 va = __builtin_bit_cast(bf16x8, av);
            if (db == 0)
                out0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[hf], out0, 0, 0, 0);
            else
                out1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[hf], out1, 0, 0, 0);
        }
    }
}

// This lane's row operand offsets (elements from a swizzled 32-row tile's row 0)
struct RowOff {
    int o[4];
};
__device__ inline RowOff row_offsets(int l32, int hh)
{
    RowOff r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r.o[c] = sw_off(l32, 2 * c + hh);
    return r;
}
__device__ inline void read_row(RowOp<true> &op, const __bf16 *tile, const RowOff &ro)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) op.x[c] = *reinterpret_cast<const bf16x8 *>(tile + ro.o[c]);
}

// A wave's 32 x 64 result (accumulators: rows channels, columns rows of the
// result) to bf16 rows of 64 channels at base + token(row) * 64.  Exchanges
// between lane halves and 16-lane rows first gather 64 consecutive bytes of a
// row in four lanes, so that a store instruction writes 16 half lines instead
// of 8-byte pieces of 32 lines.
template <typename F>
__device__ inline void store_rows(__bf16 *base, const f32x16 &o0, const f32x16 &o1, int lane, F token)
{
    // u[h][2 g + k]: channels 32 h + 8 g + 4 hh + 2 k, + 1 of row l32
    uint32_t u[2][8];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            const bf16x2 p = {static_cast<__bf16>(o0[4 * g + 2 * k]), static_cast<__bf16>(o0[4 * g + 2 * k + 1])};
            const bf16x2 q = {static_cast<__bf16>(o1[4 * g + 2 * k]), static_cast<__bf16>(o1[4 * g + 2 * k + 1])};
            u[0][2 * g + k] = __builtin_bit_cast(uint32_t, p);
            u[1][2 * g + k] = __builtin_bit_cast(uint32_t, q);
        }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        // lane halves: afterwards a lane holds whole 16-byte chunks, chunk
        // 2 x + hh of its row in u[4 x .. 4 x + 3], x = 0, 1
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const auto r = __builtin_amdgcn_permlane32_swap(u[h][4 * x + k], u[h][4 * x + 2 + k], false, false);
                u[h][4 * x + k] = r[0];
                u[h][4 * x + 2 + k] = r[1];
            }
        // 16-lane rows: lanes of rows l and l + 16 trade chunk pairs, so that
        // u[0 .. 3] belongs to row l32 & 15 and u[4 .. 7] to row 16 + (l32 & 15),
        // chunk 2 (l32 >> 4) + hh of both
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const auto r = __builtin_amdgcn_permlane16_swap(u[h][k], u[h][4 + k], false, false);
            u[h][k] = r[0];
            u[h][4 + k] = r[1];
        }
    }
    const int l16 = lane & 15, chunk = 2 * ((lane >> 4) & 1) + (lane >> 5);
    __bf16 *const r0 = base + (long long)token(l16) * kHeadDim + 8 * chunk;
    __bf16 *const r1 = base + (long long)token(16 + l16) * kHeadDim + 8 * chunk;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        *reinterpret_cast<uint4 *>(r0 + 32 * h) = make_uint4(u[h][0], u[h][1], u[h][2], u[h][3]);
        *reinterpret_cast<uint4 *>(r1 + 32 * h) = make_uint4(u[h][4], u[h][5], u[h][6], u[h][7]);
    }
}

// A wave's 32 x 64 result to fp32 rows of 64 channels, row l32 at `row` (of
// this lane's column; nullptr: not stored): 16-lane rows first gather 64
// consecutive bytes of a row in four lanes.
template <typename F>
__device__ inline void store_rows_f32(const f32x16 &o0, const f32x16 &o1, float f, int lane, F rowptr)
{
    const int l16 = lane & 15, piece = 2 * ((lane >> 4) & 1) + (lane >> 5);
    float *const p0 = rowptr(l16), *const p1 = rowptr(16 + l16);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const f32x16 &o = h ? o1 : o0;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            float a[4], b[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(f * o[8 * x + k]),
                                                                __float_as_uint(f * o[8 * x + 4 + k]), false, false);
                a[k] = __uint_as_float(r[0]);
                b[k] = __uint_as_float(r[1]);
            }
            const int ch = 32 * h + 16 * x + 4 * piece;
            if (p0) *reinterpret_cast<float4 *>(p0 + ch) = make_float4(a[0], a[1], a[2], a[3]);
            if (p1) *reinterpret_cast<float4 *>(p1 + ch) = make_float4(b[0], b[1], b[2], b[3]);
        }
    }
}

// x as a (hi, lo) pair of bf16: the rounding in the low half, the rounding of
// the rest in the high half
__device__ inline uint32_t bf16_pair(float x)
{
    const __bf16 h = static_cast<__bf16>(x);
    const __bf16 l = static_cast<__bf16>(x - static_cast<float>(h));
    return (uint32_t)__builtin_bit_cast(uint16_t, h) | ((uint32_t)__builtin_bit_cast(uint16_t, l) << 16);
}

// Sums of partial rows, one wave per output row: the terms, numbered in a
// fixed order, are dealt round-robin to NG groups of 64 / NG lanes (a lane
// takes eight channels), so NG partial rows are in flight per load.
// deal_box calls f(dx, dy, k) for the terms of an nx x ny x nk box (k
// fastest) numbered t0, t0 + 1, ... that fall to group grp, in ascending
// order; the caller advances t0 by the box's size.
template <int NG, typename F>
__device__ inline void deal_box(int nx, int ny, int nk, int grp, int t0, F f)
{
    const int nt = nx * ny * nk;
    int w = (grp - t0) & (NG - 1);   // this group's first term of the box
    int k = w % nk, dy = (w / nk) % ny, dx = (w / nk) / ny;
    for (; w < nt; w += NG) {
        f(dx, dy, k);
        k += NG;   // NG terms on
        while (k >= nk) {
            k -= nk;
            ++dy;
        }
        while (dy >= ny) {
            dy -= ny;
            ++dx;
        }
    }
}

// acc[i] += the eight floats at p (16-byte aligned), bounds-checked
__device__ inline void add8(float acc[8], const float *p, long long idx, long long lim)
{
    const uint4 p0 = ld16(p, idx, 4, lim), p1 = ld16(p, idx + 4, 4, lim);
    acc[0] += __uint_as_float(p0.x);
    acc[1] += __uint_as_float(p0.y);
    acc[2] += __uint_as_float(p0.z);
    acc[3] += __uint_as_float(p0.w);
    acc[4] += __uint_as_float(p1.x);
    acc[5] += __uint_as_float(p1.y);
    acc[6] += __uint_as_float(p1.z);
    acc[7] += __uint_as_float(p1.w);
}

// The eight groups' sums (lanes 8 grp + x hold channels 8 x ..): lanes of
// group 0 end with ((g0 + g1) + (g2 + g3)) + ((g4 + g5) + (g6 + g7)) and
// store them (split: as (hi, lo) bf16 pairs).
__device__ inline void store_group_sums(float acc[8], int grp, float *dst, long long o, long long lim, bool split = false)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float x = acc[i];
        x += __shfl_xor(x, 8);
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        acc[i] = split ? __uint_as_float(bf16_pair(x)) : x;
    }
    if (grp == 0) {
        st4f(dst, o, lim, acc[0], acc[1], acc[2], acc[3]);
        st4f(dst, o + 4, lim, acc[4], acc[5], acc[6], acc[7]);
    }
}

// The entry j of level group (qx, qy)'s 2D list that names square (u, v)
// of the same level, or -1: the inverse of list2d_entry (the square's place
// in the row-major 6x6 window around the parent, skipping the 3x3 block at
// (1 + (qx & 1), 1 + (qy & 1)); see window_slot), for squares inside the map.
__device__ inline int list2d_slot_of(int qx, int qy, int u, int v)
{
    const int au = u - (2 * (qx >> 1) - 2), av = v - (2 * (qy >> 1) - 2);
    if (au < 0 || au >= 6 || av < 0 || av >= 6) return -1;
    const int ox = 1 + (qx & 1), oy = 1 + (qy & 1);
    if (au < ox) return au * 6 + av;
    if (au < ox + 3) {
        if (av >= oy && av < oy + 3) return -1;   // the finer levels' squares
        return 6 * ox + (au - ox) * 3 + (av < oy ? av : av - 3);
    }
    return 6 * ox + 9 + (au - ox - 3) * 6 + av;
}

// Coarse-set tables in LDS (indexing the argument block with a computed
// index per lane costs scattered loads or a copy to scratch)
struct SetTab {
    int lvl[kMaxSets], M[kMaxSets], My[kMaxSets], off[kMaxSets], size[kMaxSets], woff[kMaxSets];
};
__device__ inline void load_sets(SetTab &t, const BwdArgs &a, int tid)
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

}  // namespace

}  // namespace fma_dev
