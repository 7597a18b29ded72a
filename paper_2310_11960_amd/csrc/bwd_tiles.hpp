// bwd_tiles.hpp -- what the bf16 matrix-core backward kernels share: swizzled
// 64-row tiles filled by direct-to-LDS loads, contractions over them, result
// stores and the sums of partial rows.
#pragma once

#include "bwd_device.hpp"
#include "row_groups.hpp"

namespace fma_dev {

namespace {

constexpr int ROWB = 128;          // bytes of a bf16 row of 64 channels
constexpr int TILEE = KT * 64;     // elements of one tile

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
// result) to bf16 rows of 64 channels at base + token(row) * 64.
template <typename F>
__device__ inline void store_rows(__bf16 *base, const f32x16 &o0, const f32x16 &o1, int lane, F token)
{
    const int l16 = lane & 15;
    __bf16 *const r0 = base + (long long)token(l16) * kHeadDim + 8 * store_chunk(lane);
    __bf16 *const r1 = base + (long long)token(16 + l16) * kHeadDim + 8 * store_chunk(lane);
    store_rows32(o0, 1.f, r0, r1);
    store_rows32(o1, 1.f, r0 + 32, r1 + 32);
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

}  // namespace

}  // namespace fma_dev
