// attend_route.hpp -- which kernel runs the attention of a bf16 plan: the groups
// of 128 queries (attend_group.hip), the fixed-shape stream (attend_mfma.hip)
// or the register-staged kernel (attend.hip).  Host code; the launchers and the
// plan's test export read the same rules.
#pragma once

#include "row_groups.hpp"

namespace fma_dev {

enum AttendKernel : unsigned {
    ATTEND_STAGED = 1,   // attend.hip
    ATTEND_GROUPS = 2,   // attend_group.hip
    ATTEND_STREAM = 4,   // attend_mfma.hip, a workgroup per block or cell
    ATTEND_PAIRS = 8,    // attend_mfma.hip, two cells of a map per workgroup
};

// What the groups can run: blocks that they cut into whole 32-query chunks (1D
// multiples of 32, 2D cells of 8 x 8 and 16 x 16), lists that fit the group's
// table, and under the per-level normalisation levels that fit a 32-slot piece
// (a plan without a coarse level has none, whatever its slots per level).
inline bool group_fits(const AttnArgs &a, bool two_d)
{
    if (a.n > 0x7fffffffLL - 4096 || a.qbar) return false;
    if (a.norm_level && a.nslot > 0 && a.slot_group > 32) return false;
    if (!two_d) return a.r % 32 == 0 && group_lists_fit<GEOM_1D>(a);
    return a.r == 8 ? group_lists_fit<GEOM_2DP>(a) : a.r == 16 && group_lists_fit<GEOM_2D>(a);
}

// The kernel of a plan; ATTEND_GROUPS | ATTEND_STREAM where it depends on how
// the call fills the device (groups_win); 0: none (fma_plan makes no such plan).
//
// Groups are the faster kernel for head dims 32 and 128 and blocks of 32
// against the register-staged one (d = 128 causal 7808 x 128, 64 slices: 581 ->
// 149 us; blocks of 32, 64 slices of 4000: 207 -> 42 us), and at d = 64 against
// the stream for every 2D map (128 x 128 at 32 slices 163 -> 141 us, 16 x 16
// cells 418 -> 322, 120 x 168 per level 272 -> 233), 1D blocks of 64 (48 slices
// of 16384: 150 -> 111 us, causal 128 -> 89), causal blocks of 192 (169 -> 126)
// and causal blocks of 128, half of whose near tiles are partly masked (108 ->
// 102; 8 slices of 4096 11.6 -> 10.1).
inline unsigned attend_kernels(const AttnArgs &a, bool two_d)
{
    if (group_fits(a, two_d))
        return two_d || a.head_dim != kHeadDim || a.r < 128 || (a.causal && a.r < 256) ? ATTEND_GROUPS
                                                                                        : ATTEND_GROUPS | ATTEND_STREAM;
    if (a.head_dim != kHeadDim || (two_d ? a.r < 8 : a.r < 64)) return ATTEND_STAGED;
    if (a.nslot > kMaxSlotTable) return 0;
    if (a.qbar) return a.nslot > 0 && !a.norm_level && a.rank == 1 ? ATTEND_STREAM : 0;   // FMA-linear
    if (!two_d) return a.r >= 128 ? ATTEND_STREAM : 0;
    if (!a.norm_level || a.nslot == 0) return 0;   // joint normalisation on maps: groups
    return pair_cells_2d(a.r, a.nby, a.nslot, a.slot_group) ? ATTEND_PAIRS : ATTEND_STREAM;
}

// 1D blocks of 128 and 256 and bidirectional ones of 192 at d = 64, on a device
// of `cus` CUs.  Both kernels do the same arithmetic; what differs is how they
// fill the device.  A group has four waves, one per SIMD of its CU, and four
// fit a CU; the stream's workgroup is a whole block (eight waves for 256) that
// loads the near window once, and its grid is cut evenly among the eight XCDs
// only if the blocks are a multiple of eight (306 groups of blocks of 256: 23.7
// us against 32.4).
//   256: up to one group per CU the groups use twice the CUs (256 groups 19.8 us
//     against 20.9, causal 15.0 against 17.3), and so does the remainder when
//     the last of several such rounds is the half that the stream would leave
//     empty (576: 28.9 / 31.2, causal 22.6 / 24.5; 768: 31.4 / 32.1); whole
//     rounds of the stream beat them (512: 24.5 / 21.8, causal 18.6 / 18.0;
//     1024: 39.5 / 34.8, causal 29.0 / 26.5).
//   128: the same number of workgroups; the groups start faster (256: 12.4 / 13.0,
//     512: 16.1 / 16.3), past two per CU the persistent stream catches up (640:
//     19.9 / 19.5, 1024: 26.4 / 25.8).
//   More than one round of groups: the stream (65536 x 128, 16 slices 180 / 175
//     us; blocks of 256 287 / 261).
//   192: groups straddle blocks, and the stream's six waves leave a quarter of
//     the device idle; groups win once the stream needs more than three
//     workgroups per CU (1536 groups 52 / 64 us, 48 slices of 16384 185 / 214;
//     384: 22.9 / 19.4, 1152: 44.4 / 41.0).
inline bool groups_win(const AttnArgs &a, int cus)
{
    const long long groups = (long long)a.nslice * row_groups<GEOM_1D>(a);
    const long long blocks = (long long)a.nslice * a.tiles_per_slice;
    if (a.r % 128) return blocks > 3LL * cus;
    if (groups > 4LL * cus) return false;
    if (blocks % 8) return true;
    return a.r == 128 ? groups <= 2LL * cus : (groups + cus - 1) / cus % 2 == 1;
}

}  // namespace fma_dev
