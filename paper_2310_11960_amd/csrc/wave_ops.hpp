// wave_ops.hpp -- exchanges between the lanes of a wave that the bf16 kernels
// share: the two halves of a 32x32 accumulator's columns, and the 64-byte
// pieces in which results leave.
#pragma once

#include "fma_device.hpp"

namespace fma_dev {

namespace {

// max / sum of x over this lane and lane ^ 32 (v_permlane32_swap: a VALU
// exchange of the wave's halves, no LDS round trip)
__device__ __attribute__((always_inline)) inline float pair_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __attribute__((always_inline)) inline float pair_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// two floats as a pair of bf16, lo in the low half
__device__ __attribute__((always_inline)) inline uint32_t pack_bf16(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 p = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, p);
}

// One 32-channel accumulator packed to bf16 pairs, u[2 g + k] channels 8 g +
// 4 (lane >> 5) + 2 k, + 1 of row lane & 31, rearranged for 16-byte stores of
// which four lanes cover 64 consecutive bytes: afterwards u[0 .. 3] belong to
// row lane & 15 and u[4 .. 7] to row 16 + (lane & 15), both channels 8 c .. of
// chunk c = store_chunk(lane).  A store instruction then writes 16 half lines
// instead of 8-byte pieces of 32 lines.
__device__ __attribute__((always_inline)) inline void gather_rows(uint32_t (&u)[8])
{
    // lane halves: whole 16-byte chunks, chunk 2 x + (lane >> 5) in u[4 x .. 4 x + 3]
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const auto r = __builtin_amdgcn_permlane32_swap(u[4 * x + k], u[4 * x + 2 + k], false, false);
            u[4 * x + k] = r[0];
            u[4 * x + 2 + k] = r[1];
        }
    // 16-lane rows trade chunk pairs
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const auto r = __builtin_amdgcn_permlane16_swap(u[k], u[4 + k], false, false);
        u[k] = r[0];
        u[4 + k] = r[1];
    }
}
__device__ inline int store_chunk(int lane) { return 2 * ((lane >> 4) & 1) + (lane >> 5); }

// One 32-channel accumulator (rows channels, columns rows of the result;
// scaled by f) to bf16 rows: row lane & 15 at r0, row 16 + (lane & 15) at r1
// (both at this lane's chunk, 8 * store_chunk(lane) elements into the 32).
__device__ __attribute__((always_inline)) inline void store_rows32(const f32x16 &o, float f, __bf16 *r0, __bf16 *r1)
{
    uint32_t u[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) u[x] = pack_bf16(o[2 * x] * f, o[2 * x + 1] * f);
    gather_rows(u);
    *reinterpret_cast<uint4 *>(r0) = make_uint4(u[0], u[1], u[2], u[3]);
    *reinterpret_cast<uint4 *>(r1) = make_uint4(u[4], u[5], u[6], u[7]);
}

}  // namespace

}  // namespace fma_dev
