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

}  // namespace

extern "C" {

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
