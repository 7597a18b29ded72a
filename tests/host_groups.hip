// Host build of the index and dispatch rules of the group kernels (test
// infrastructure, no device code): plans come in as the values that
// fma_plan_params writes.
#include <stdint.h>
#include <string.h>

#include "attend_route.hpp"

using namespace fma_dev;

namespace {

// The attention's arguments of a plan (fma_plan_params' order), as far as the
// rules read them.
AttnArgs args_of(const int64_t *v)
{
    AttnArgs a;
    memset(&a, 0, sizeof(a));
    a.n = v[0];
    a.side = (int)v[1];
    a.r = (int)v[2];
    a.nbx = (int)v[3];
    a.qtile = (int)v[4];
    a.tiles_per_slice = (int)v[5];
    a.nslice = (int)v[6];
    a.R = (int)v[7];
    a.causal = (int)v[8];
    a.nslot = (int)v[9];
    a.slot_group = (int)v[10];
    a.rank = (int)v[11];
    a.norm_level = (int)v[12];
    a.lv.nlev = (int)v[18];
    a.nby = (int)v[38];
    a.head_dim = (int)v[40];
    static const char linear = 0;
    if (v[33] && a.lv.nlev > 0) a.qbar = &linear;   // only compared with nullptr
    for (int e = 0; e < a.lv.nlev && e < kMaxSets; ++e) {
        const int64_t *s = v + 41 + 6 * e;
        a.lv.off[e] = (int)s[0];
        a.lv.M[e] = (int)s[1];
        a.lv.My[e] = (int)s[2];
        a.lv.size[e] = (int)s[3];
        a.lv.woff[e] = (int)s[4];
        a.lv.lvl[e] = (int)s[5];
    }
    return a;
}

int geometry(const int64_t *v) { return v[13] == 1 ? GEOM_1D : v[2] == 8 ? GEOM_2DP : GEOM_2D; }

// The rows of one wave of a group as the kernels walk them: every loaded row
// (its smallest and largest token), the taken 32-row pieces in order, the
// wave's own rows.  TR > 0: the attention's tiles of TR rows; 0: the backward's
// runs of eight in tiles of 64, of the queries' window or (KEYS) the keys'.
template <int GEOM, int TR, bool KEYS>
void walk(const AttnArgs &a, int g, int wave, int64_t *out)
{
    const RowGroup m = row_group<GEOM, KEYS>(a, g, wave);
    int64_t taken = 0, diag = -1, lo = a.n, hi = -1, *rows = out + 6 + 32;
    constexpr int T = TR > 0 ? TR : 64, PPT = T / 32;
    for (int t = 0; t < (m.npiece + PPT - 1) / PPT; ++t) {
        int64_t tok[T];
        if constexpr (TR > 0) {
            const TileCell cell = tile_cell<GEOM, T>(a, m, t);
            for (int r = 0; r < T; ++r) tok[r] = tile_token<GEOM, T>(a, m, cell, t, r);
        } else {
            for (int r = 0; r < T; ++r) tok[r] = window_run<GEOM>(a, m, 8 * t + r / 8) + r % 8;
        }
        for (int r = 0; r < T; ++r) {
            lo = tok[r] < lo ? tok[r] : lo;
            hi = tok[r] > hi ? tok[r] : hi;
        }
        for (int hb = 0; hb < PPT; ++hb) {
            const int p = PPT * t + hb;
            if ((TR > 0 && p >= m.npiece) || !piece_used<GEOM>(a, m, p)) continue;
            if (GEOM == GEOM_1D && 32 * p == m.wdiag) diag = taken;
            for (int r = 0; r < 32; ++r) rows[taken++] = tok[32 * hb + r];
        }
    }
    out[0] = m.active;
    out[1] = m.blk;
    out[2] = taken;
    out[3] = diag;
    out[4] = lo;
    out[5] = hi;
    for (int r = 0; r < 32; ++r) out[6 + r] = m.active ? wave_token<GEOM>(a, m, m.pos0 + r) : -1;
}

template <int GEOM>
void walk_kind(const AttnArgs &a, int kind, int g, int wave, int64_t *out)
{
    switch (kind) {
    case 0: return walk<GEOM, 64, false>(a, g, wave, out);
    case 1: return walk<GEOM, 32, false>(a, g, wave, out);
    case 2: return walk<GEOM, 0, false>(a, g, wave, out);
    default: return walk<GEOM, 0, true>(a, g, wave, out);
    }
}

// A group's list table: its sizes and the wave's part, then every row's coarse
// row (-1: empty) and whether the wave's cell sees it.
template <int GEOM, bool PL>
void list_table(const AttnArgs &a, int g, int wave, int64_t *out)
{
    const RowGroup m = row_group<GEOM, false>(a, g, wave);
    const GroupLists l = group_lists<GEOM, PL>(a, m, g, wave);
    out[0] = l.npiece;
    out[1] = l.pc0;
    out[2] = l.npc;
    out[3] = l.npc > 0 ? list_table_rows(l) : 0;
    out[4] = m.blk;
    for (int e = 0; e < out[3]; ++e) {
        int mask;
        out[5 + 2 * e] = list_row<GEOM, PL>(a, m, l, g, a.lv, e, mask);
        out[6 + 2 * e] = (mask >> (GEOM == GEOM_2DP && !PL ? wave >> 1 : 0)) & 1;
    }
}

template <bool TWO_D>
void sibling(const AttnArgs &a, int gslot, int grp, int64_t *out)
{
    const SiblingGroup s = sibling_group<TWO_D>(a, grp);
    const int nchunk = s.ncx * s.ncy * s.cpb;
    out[0] = s.cx0;
    out[1] = s.cy0;
    out[2] = nchunk;
    int64_t *o = out + 3;
    for (int slot = 0; slot < gslot; ++slot) {
        int mask;
        *o++ = sibling_slot<TWO_D>(a, s, gslot, slot, mask);
        *o++ = mask;
    }
    for (int c = 0; c < nchunk; ++c) {
        int i, j, p;
        sibling_block(s, c, i, j, p);
        *o++ = i;
        *o++ = j;
        for (int r = 0; r < 32; ++r) *o++ = sibling_run<TWO_D>(a, s, c, r / 8) + r % 8;
    }
}

}  // namespace

extern "C" {

int64_t host_group_count(const int64_t *plan)
{
    const AttnArgs a = args_of(plan);
    const int geom = geometry(plan);
    return geom == GEOM_1D ? row_groups<GEOM_1D>(a) : geom == GEOM_2DP ? row_groups<GEOM_2DP>(a) : row_groups<GEOM_2D>(a);
}

void host_group_walk(const int64_t *plan, int kind, int g, int wave, int64_t *out)
{
    const AttnArgs a = args_of(plan);
    switch (geometry(plan)) {
    case GEOM_1D: return walk_kind<GEOM_1D>(a, kind, g, wave, out);
    case GEOM_2DP: return walk_kind<GEOM_2DP>(a, kind, g, wave, out);
    default: return walk_kind<GEOM_2D>(a, kind, g, wave, out);
    }
}

void host_group_lists(const int64_t *plan, int pl, int g, int wave, int64_t *out)
{
    const AttnArgs a = args_of(plan);
    switch (geometry(plan)) {
    case GEOM_1D: return pl ? list_table<GEOM_1D, true>(a, g, wave, out) : list_table<GEOM_1D, false>(a, g, wave, out);
    case GEOM_2DP: return pl ? list_table<GEOM_2DP, true>(a, g, wave, out) : list_table<GEOM_2DP, false>(a, g, wave, out);
    default: return pl ? list_table<GEOM_2D, true>(a, g, wave, out) : list_table<GEOM_2D, false>(a, g, wave, out);
    }
}

int host_sibling_slots(const int64_t *plan)
{
    return group_slots(plan[13] == 2, (int)plan[11], (int)plan[18]);
}

void host_sibling_group(const int64_t *plan, int grp, int64_t *out)
{
    const AttnArgs a = args_of(plan);
    if (plan[13] == 2) sibling<true>(a, host_sibling_slots(plan), grp, out);
    else sibling<false>(a, host_sibling_slots(plan), grp, out);
}

unsigned host_attend_kernels(const int64_t *plan) { return attend_kernels(args_of(plan), plan[13] == 2); }

// launch_backward on arguments whose sibling groups say that the bf16 streamed
// query pass runs: its status.  tokens: per slice; launches nothing where the
// blocks do not stream.
int host_backward_status(int64_t tokens, int ngrp)
{
    BwdArgs a;
    memset(&a, 0, sizeof(a));
    a.n = tokens;
    a.r = a.qtile = 64;
    a.nslice = a.heads = a.heads_w = a.pslices = a.rank = 1;
    a.nblocks = a.nbx = (int)(tokens / 64);
    a.nby = 1;
    a.ngrp = ngrp;
    a.gslot = 6;
    a.nslot = 3;
    a.R = 4;
    a.lv.nlev = 1;
    return (int)launch_backward(a, true, false, nullptr);
}

int host_groups_win(const int64_t *plan, int cus) { return groups_win(args_of(plan), cus); }

}  // extern "C"
