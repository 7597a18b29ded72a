// level_weights.hpp -- the printed per-level normalisation of one 32-key block
// of coarse scores.
#pragma once

#include "wave_ops.hpp"

namespace fma_dev {

namespace {

// Printed per-level normalisation of one 32-key block of coarse scores x
// (log2 units, masked slots -inf): the keys form aligned groups of grp (4, 8,
// 16 or 32) slots, one level each; element i of a lane holds key row
// 8 * (i >> 2) + 4 * hh + (i & 3), so a group is 1 chunk of 4 in-lane (grp 4),
// that chunk in both lanes of the pair lane, lane ^ 32 (8), two chunks (16) or
// all four (32).  Each key's weight becomes lnear * exp2(x - m_g) / l_g, with
// m_g and l_g the group's own maximum and sum; an empty group gives 0.
__device__ __attribute__((always_inline)) inline void level_weights(f32x16 &x, float lnear, int grp)
{
    float cm[4], cl[4];
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
        for (int e = 0; e < 4; ++e) x[4 * c + e] = __builtin_amdgcn_exp2f(x[4 * c + e] - cm[c]);
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
        const float f = cl[c] > 0.0f ? lnear / cl[c] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * c + e] *= f;
    }
}

}  // namespace

}  // namespace fma_dev
