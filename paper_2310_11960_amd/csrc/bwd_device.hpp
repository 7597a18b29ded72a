// bwd_device.hpp -- helpers shared by the backward kernels (gfx950): checked
// global accesses, matrix-core operands and contractions over swizzled LDS
// tiles, the base blocks' geometry and the interaction-list sources.
#pragma once

#include "fma_device.hpp"
#include "fma_kernels.hpp"
#include "wave_ops.hpp"

namespace fma_dev {

namespace {

constexpr int KT = 64;     // rows per tile
constexpr int PB = 72;     // LDS pitch (bf16 elements) of 64-entry rows
constexpr int PF = 68;     // LDS pitch (fp32 elements) of 64-entry rows
constexpr int PQB = 40;    // LDS pitch (bf16) of 32-entry transposed rows
constexpr int PQF = 36;    // LDS pitch (fp32) of 32-entry transposed rows
constexpr int kMaxSlots = 448;   // interaction-list slots a plan may have

template <bool BF16>
struct Elt;
template <>
struct Elt<true> {
    typedef __bf16 T;
    static constexpr int P = PB, PQ = PQB, PER16 = 8;   // elements per 16-byte chunk
};
template <>
struct Elt<false> {
    typedef float T;
    static constexpr int P = PF, PQ = PQF, PER16 = 4;
};

// ------------------------------------------------------------- checked memory
__device__ inline uint4 ld16(const void *base, long long elem, int esize, long long lim)
{
    // 16 bytes starting at element `elem` (a multiple of 16 / esize)
    if (elem < 0 || elem + 16 / esize > lim) return make_uint4(0, 0, 0, 0);
    return *reinterpret_cast<const uint4 *>(static_cast<const char *>(base) + elem * esize);
}

__device__ inline float ldf(const float *p, long long i, long long lim) { return (i >= 0 && i < lim) ? p[i] : 0.f; }

__device__ inline void stf(float *p, long long i, long long lim, float x)
{
    if (i >= 0 && i < lim) p[i] = x;
}

__device__ inline void st4f(float *p, long long i, long long lim, float a, float b, float c, float d)
{
    if (i >= 0 && i + 4 <= lim) *reinterpret_cast<float4 *>(p + i) = make_float4(a, b, c, d);
}

// 4 consecutive output elements of the I/O dtype
template <bool BF16>
__device__ inline void st4(void *base, long long i, long long lim, float a, float b, float c, float d)
{
    if (i < 0 || i + 4 > lim) return;
    if constexpr (BF16)
        *reinterpret_cast<uint2 *>(static_cast<__bf16 *>(base) + i) = make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
    else
        *reinterpret_cast<float4 *>(static_cast<float *>(base) + i) = make_float4(a, b, c, d);
}

__device__ inline float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ inline int acc_row(int i, int hh) { return 8 * (i >> 2) + 4 * hh + (i & 3); }

// ------------------------------------------------------------- operands
// A row operand: this lane's part of one 64-channel row (lane & 31 = row,
// lane >> 5 = which channels), as the A or the B side of a 32x32 MFMA.
template <bool BF16>
struct RowOp;
template <>
struct RowOp<true> {
    bf16x8 x[4];   // channels 16 c + 8 hh .. + 7
    __device__ void from_lds(const __bf16 *row, int hh)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = *reinterpret_cast<const bf16x8 *>(row + 16 * c + 8 * hh);
    }
    __device__ float chan(int c, int e) const { return static_cast<float>(x[c][e]); }
};
template <>
struct RowOp<false> {
    float x[32];   // channel 2 c + hh
    __device__ void from_lds(const float *row, int hh)
    {
#pragma unroll
        for (int c = 0; c < 32; ++c) x[c] = row[2 * c + hh];
    }
};

// acc[m][n] += sum over the 64 channels of A[m][ch] B[n][ch]
template <bool BF16>
__device__ inline f32x16 contract_channels(const RowOp<BF16> &A, const RowOp<BF16> &B, f32x16 acc)
{
    if constexpr (BF16) {
#pragma unroll
        for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.x[c], B.x[c], acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int c = 0; c < 32; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A.x[c], B.x[c], acc, 0, 0, 0);
    }
    return acc;
}

// out_db[ch][n] += sum over 32 rows r of T[ch][rowbase + r] w[r][n], for
// ch = 32 db + (lane & 31); w in accumulator layout (column n = lane & 31).
template <bool BF16>
__device__ inline void contract_rows(const typename Elt<BF16>::T *T, int pitch, int rowbase, const f32x16 &w, int l32,
                                     int hh, f32x16 &out0, f32x16 &out1)
{
    if constexpr (BF16) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            bf16x8 pb;
#pragma unroll
            for (int e = 0; e < 8; ++e) pb[e] = static_cast<__bf16>(w[8 * hf + e]);
            const int base = rowbase + 16 * hf + 4 * hh;
#pragma unroll
            for (int db = 0; db < 2; ++db) {
                const __bf16 *t = T + (db * 32 + l32) * pitch + base;
                const bf16x4 lo = *reinterpret_cast<const bf16x4 *>(t);
                const bf16x4 hi = *reinterpret_cast<const bf16x4 *>(t + 8);
                const bf16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                if (db == 0)
                    out0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pb, out0, 0, 0, 0);
                else
                    out1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pb, out1, 0, 0, 0);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = rowbase + acc_row(i, hh);
            out0 = __builtin_amdgcn_mfma_f32_32x32x2f32(T[l32 * pitch + row], w[i], out0, 0, 0, 0);
            out1 = __builtin_amdgcn_mfma_f32_32x32x2f32(T[(32 + l32) * pitch + row], w[i], out1, 0, 0, 0);
        }
    }
}

// bf16 tiles in LDS: 64-channel rows of 128 bytes whose 16-byte chunk c sits
// at chunk c ^ swz(row).  For the row reads of a 32x32 operand (ds_read_b128,
// lane = row) the rows of any 16 lanes land in distinct bank groups, and for
// the transposing reads (ds_read_b64_tr_b16, four rows of four chunks per 16
// lanes) rows r and r + 2 sit in opposite 64-byte halves, so neither kind
// conflicts; fp32 tiles keep the padded pitch.
__device__ inline int swz(int row) { return (2 * (row & 3)) ^ ((row >> 2) & 1) ^ (2 * ((row >> 3) & 1)); }
__device__ inline int sw_off(int row, int chunk) { return row * kHeadDim + 8 * (chunk ^ swz(row)); }

// this lane's part of row `row` of a swizzled bf16 tile (as RowOp::from_lds)
__device__ inline void row_from_tile(RowOp<true> &op, const __bf16 *tile, int row, int hh)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) op.x[c] = *reinterpret_cast<const bf16x8 *>(tile + sw_off(row, 2 * c + hh));
}

// contract_rows on a swizzled bf16 tile read with transposing loads: the A
// operand of lane (l32, hh) is channel 32 db + l32 at rows rowbase + 16 hf +
// {4 hh .. 4 hh + 3, 8 + 4 hh .. 8 + 4 hh + 3}, the order of the B operand's
// k slots.  Lanes 16 g + 4 j + q read rows 4 (g >> 1) + j (and + 8), chunk
// 4 db + 2 (g & 1) + (q >> 1), half q & 1.
__device__ inline void contract_rows_tr(const __bf16 *tile, int rowbase, const f32x16 &w, int lane, f32x16 &out0,
                                        f32x16 &out1)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const int gq = lane >> 4, s4 = lane & 15, j = s4 >> 2, q = s4 & 3;
    const int row = 4 * (gq >> 1) + j;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        bf16x8 pb;
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[e] = static_cast<__bf16>(w[8 * hf + e]);
        const __bf16 *t16 = tile + (rowbase + 16 * hf) * kHeadDim;
#pragma unroll
        for (int db = 0; db < 2; ++db) {
            const int chunk = 4 * db + 2 * (gq & 1) + (q >> 1);
            const s16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_s16x4 *)(t16 + sw_off(row, chunk) + 4 * (q & 1)));
            const s16x4 r2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_s16x4 *)(t16 + sw_off(row + 8, chunk) + 4 * (q & 1)));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            const s16x8 av = {r1[0], r1[1], r1[2], r1[3], r2[0], r2[1], r2[2], r2[3]};
            const bf16x8 va = __builtin_bit_cast(bf16x8, av);
            if (db == 0)
                out0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, out0, 0, 0, 0);
            else
                out1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, out1, 0, 0, 0);
        }
    }
}

// One channel half db of contract_rows_tr (rows 0..31 of the tile), with the
// B operand given as bf16: pb[hf] holds w's entries 8 hf .. 8 hf + 7.
__device__ inline f32x16 contract_rows_tr1(const __bf16 *tile, const bf16x8 pb[2], int lane, int db, f32x16 out)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const int gq = lane >> 4, s4 = lane & 15, j = s4 >> 2, q = s4 & 3;
    const int row = 4 * (gq >> 1) + j;
    const int chunk = 4 * db + 2 * (gq & 1) + (q >> 1);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const __bf16 *t16 = tile + (16 * hf) * kHeadDim;
        const s16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + sw_off(row, chunk) + 4 * (q & 1)));
        const s16x4 r2 =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + sw_off(row + 8, chunk) + 4 * (q & 1)));
        const s16x8 av = {r1[0], r1[1], r1[2], r1[3], r2[0], r2[1], r2[2], r2[3]};
        out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), pb[hf], out, 0, 0, 0);
    }
    return out;
}

// Per-level softmax of one 32-slot block of scores (per-level
// normalisation): the slots form aligned groups of grp (4, 8, 16 or 32)
// rows, one level each.  x holds the lane's scaled scores (log2 units, -inf
// for empty slots) in accumulator layout (element i is row acc_row(i, hh)),
// so a group of 4 is one chunk of 4 elements, 8 that chunk in both halves of
// the wave (lane ^ 32), 16 two chunks and 32 all four.  On return x holds
// dS = P (dP - D_g) with P = exp2(x - m_g) / l_g; lse[c] = m_g + log2 l_g
// (-inf for an empty group) and dg[c] = D_g = sum_g P dP of the group of
// chunk c.
__device__ inline void level_block(f32x16 &x, const f32x16 &dp, int grp, float (&lse)[4], float (&dg)[4])
{
    float cm[4], cl[4], cd[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) cm[c] = fmaxf(fmaxf(x[4 * c], x[4 * c + 1]), fmaxf(x[4 * c + 2], x[4 * c + 3]));
    if (grp >= 16) {
        cm[0] = cm[1] = fmaxf(cm[0], cm[1]);
        cm[2] = cm[3] = fmaxf(cm[2], cm[3]);
    }
    if (grp >= 32) cm[0] = cm[1] = cm[2] = cm[3] = fmaxf(cm[0], cm[2]);
    if (grp >= 8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) cm[c] = pair_max(cm[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        cm[c] = cm[c] > -INFINITY ? cm[c] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] = fexp2(x[4 * c + e] - cm[c]);
        cl[c] = (x[4 * c] + x[4 * c + 1]) + (x[4 * c + 2] + x[4 * c + 3]);
    }
    if (grp >= 16) {
        cl[0] = cl[1] = cl[0] + cl[1];
        cl[2] = cl[3] = cl[2] + cl[3];
    }
    if (grp >= 32) cl[0] = cl[1] = cl[2] = cl[3] = cl[0] + cl[2];
    if (grp >= 8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) cl[c] = pair_sum(cl[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float inv = cl[c] > 0.0f ? 1.0f / cl[c] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] *= inv;
        cd[c] = (x[4 * c] * dp[4 * c] + x[4 * c + 1] * dp[4 * c + 1]) +
                (x[4 * c + 2] * dp[4 * c + 2] + x[4 * c + 3] * dp[4 * c + 3]);
    }
    if (grp >= 16) {
        cd[0] = cd[1] = cd[0] + cd[1];
        cd[2] = cd[3] = cd[2] + cd[3];
    }
    if (grp >= 32) cd[0] = cd[1] = cd[2] = cd[3] = cd[0] + cd[2];
    if (grp >= 8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) cd[c] = pair_sum(cd[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] *= dp[4 * c + e] - cd[c];
        lse[c] = cl[c] > 0.0f ? cm[c] + __log2f(cl[c]) : -INFINITY;
        dg[c] = cd[c];
    }
}

// token of position p (0 .. qtile-1) of block b
template <bool TWO_D>
__device__ inline long long block_tok(const BwdArgs &a, int b, int p)
{
    if constexpr (TWO_D) {
        const int cx = b / a.nby, cy = b - (b / a.nby) * a.nby;
        return (long long)(cx * a.r + p / a.r) * a.side + cy * a.r + p % a.r;
    } else {
        return (long long)b * a.r + p;
    }
}

// --------------------------------------------------------------- tiles
// 2D: the in-map 3x3 neighbourhood of a cell is a rectangle of cells, walked
// row-major (the forward's order); near cell ci is cell (x0 + ci / ny,
// y0 + ci % ny).
struct Near2D {
    int x0, y0, ny, ncell;
};

__device__ inline Near2D near2d(const BwdArgs &a, int b)
{
    const int cx = b / a.nby, cy = b - (b / a.nby) * a.nby;
    Near2D d;
    d.x0 = cx > 0 ? cx - 1 : 0;
    d.y0 = cy > 0 ? cy - 1 : 0;
    const int x1 = cx + 1 < a.nbx ? cx + 1 : cx, y1 = cy + 1 < a.nby ? cy + 1 : cy;
    d.ny = y1 - d.y0 + 1;
    d.ncell = (x1 - d.x0 + 1) * d.ny;
    return d;
}

// token of position p (row-major in the r x r cell, lg = log2 r) of near cell ci
__device__ inline long long near2d_token(const BwdArgs &a, const Near2D &d, int ci, int p, int lg)
{
    const int qx = ci / d.ny;
    const int ux = d.x0 + qx, uy = d.y0 + ci - qx * d.ny;
    return (long long)((ux << lg) + (p >> lg)) * a.side + (uy << lg) + (p & (a.r - 1));
}

// Coarse row of interaction-list slot `slot` of block b, or -1 for an empty
// slot.  Joint layout: slot = set * K + j; per-level layout: slot = level *
// slot_group + basis * K + j (slots past a level's rank * K are padding).
template <bool TWO_D>
__device__ inline int coarse_source(const BwdArgs &a, int b, int slot)
{
    constexpr int K = TWO_D ? kSlots2D : kSlots1D;
    if (slot >= a.nslot) return -1;
    int set, j;
    if (a.norm_level) {
        const int lev = slot / a.slot_group, rem = slot - lev * a.slot_group;
        const int basis = rem / K;
        if (basis >= a.rank) return -1;
        set = lev * a.rank + basis;
        j = rem - basis * K;
    } else {
        set = slot / K;
        j = slot - set * K;
    }
    if (set >= a.lv.nlev) return -1;
    int g;
    if constexpr (TWO_D)
        g = list2d_entry(b / a.nby, b % a.nby, a.lv.lvl[set], j, a.lv.M[set], a.lv.My[set]);
    else
        g = list1d_entry(b, a.lv.lvl[set], j, a.lv.M[set], a.causal);
    return g < 0 ? -1 : a.lv.off[set] + g;
}

}  // namespace

}  // namespace fma_dev
