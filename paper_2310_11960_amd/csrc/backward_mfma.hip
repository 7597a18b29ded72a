// backward_mfma.hip -- the bf16 backward on streams of direct-to-LDS tiles
// (see backward.hip for the method and row_groups.hpp for the groups of rows,
// their windows and lists).
#include "bwd_tiles.hpp"

namespace fma_dev {

namespace {

// ---------------------------------------------------------------- query pass
// Gradients of the queries: the near window's keys and the interaction-list
// rows, with the softmax's reference maximum and sum formed on the way
// (dq = sum exp2(s - m)(dP - D) k, dQ = tau dq / l at the end), and lse, D of
// every query for the other passes.
//
// Bounds, at 1D 65536 x 128, 32 slices: it reads Q, K, V, O, dO and writes dQ
// once, 1.6 GB (310 us at a copy's 5.2 TB/s).  The coarse rows' gradients are
// a pass of their own (bwd_coarse_mfma): kept in this kernel, they needed the
// queries' transposes in LDS (61 KB a workgroup, two waves per SIMD) and four
// barriers per 32 slots.  With them apart, 37 KB and three waves per SIMD.
// Query pass with the coarse pass and the reduction of its partial rows:
// 1D 65536 x 128 918 -> 711 us, causal 16384 x 128 (96 slices) 591 -> 486 us,
// 128 x 128 map (128 slices) 2890 -> 1119 us, blocks of 32 (64 slices of
// 4000) 296 -> 98 us.
struct QuerySmem {
    __bf16 k[2][TILEE];
    __bf16 v[2][TILEE];
    ListSmem list;
    SetTab st;
};

template <int GEOM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void bwd_query_mfma(BwdArgs a)
{
    constexpr bool TWO_D = GEOM != GEOM_1D;
    __shared__ __attribute__((aligned(16))) QuerySmem sm;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int gps = (int)row_groups<GEOM>(a);
    const int slice = __builtin_amdgcn_readfirstlane((int)(id / (unsigned)gps));
    const int grp = (int)(id - (unsigned)slice * (unsigned)gps);
    const RowGroup m = row_group<GEOM, false>(a, grp, wave);
    load_sets(sm.st, a, tid);

    const char *const kg = static_cast<const char *>(a.k) + (long long)slice * a.n * ROWB;
    const char *const vg = static_cast<const char *>(a.v) + (long long)slice * a.n * ROWB;
    const char *const kb = static_cast<const char *>(a.kbar) + (long long)slice * a.R * ROWB;
    const char *const vb = static_cast<const char *>(a.vbar) + (long long)slice * a.R * ROWB;
    const int loff = dma_lane_off(lane, wave & 1);

    const GroupLists gl = group_lists<GEOM>(a, m, grp);
    const int nnear = (m.npiece + 1) / 2, nct = (gl.npiece + 1) / 2;   // near and coarse tiles

    // Tile t into stage st: wave w loads rows 8 w .. and 8 (w + 4) .. of K and V
    auto issue = [&](int t, int st) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int i = wave + 4 * jj;
            const uint32_t kd = lds_u32(sm.k[st]) + i * 1024, vd = lds_u32(sm.v[st]) + i * 1024;
            if (t < nnear) {
                const long long o = window_run<GEOM>(a, m, 8 * t + i) * ROWB + loff;
                dma16(kg + o, kd);
                dma16(vg + o, vd);
            } else {
                // gathered rows (a piece without rows, which no wave takes: row 0)
                const int row = sm.list.crow[(t - nnear) * KT + 8 * i + (lane >> 3)];
                const long long o = (long long)(row < 0 ? 0 : row) * ROWB + loff - (lane >> 3) * ROWB;
                dma16(kb + o, kd);
                dma16(vb + o, vd);
            }
        }
    };
    issue(0, 0);

    // this lane's query and its upstream gradient, D = dO . O
    const long long qtok = m.active ? wave_token<GEOM>(a, m, m.pos0 + l32) : 0;
    const long long qrow = ((long long)slice * a.n + qtok) * kHeadDim;
    RowOp<true> qo, go;
    float dpart = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        qo.x[c] = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(a.q) + qrow + 16 * c + 8 * hh);
        go.x[c] = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(a.dout) + qrow + 16 * c + 8 * hh);
        const bf16x8 o = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(a.out) + qrow + 16 * c + 8 * hh);
#pragma unroll
        for (int e = 0; e < 8; ++e) dpart += static_cast<float>(go.x[c][e]) * static_cast<float>(o[e]);
    }
    const float dd = pair_sum(dpart);
    __syncthreads();   // the set tables
    build_lists<GEOM>(a, m, gl, grp, sm.st, wave, lane, sm.list);

    const float cs = a.scale_log2;
    const float off = cs < 0.f ? INFINITY : -INFINITY;   // a masked score: -inf once scaled
    const RowOff ro = row_offsets(l32, hh);
    const TrOff to = tr_offsets(lane);
    f32x16 dq0 = {0}, dq1 = {0};
    float mrun = 0.f, lrun = 0.f;
    bool first = true;
    // one 32-row piece; mode 0: every row visible, 1: causal diagonal (row <=
    // query), 2: rows whose bit 8 (i >> 2) + (i & 3) of mw is set
    auto piece = [&](const __bf16 *kt, const __bf16 *vt, int mode, uint32_t mw) {
        RowOp<true> rop;
        read_row(rop, kt, ro);
        f32x16 s = contract_channels<true>(rop, qo, f32x16{0});   // S^T: keys x queries
        __builtin_amdgcn_sched_barrier(0);
        read_row(rop, vt, ro);
        f32x16 dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) dp[i] = -dd;
        dp = contract_channels<true>(rop, go, dp);                // dP^T - D
        __builtin_amdgcn_sched_barrier(0);
        auto mask_rows = [&](f32x16 &x) {
            if (mode == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = acc_row(i, hh) <= l32 ? x[i] : off;
            } else if (mode == 2) {
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = (mw >> (8 * (i >> 2) + (i & 3))) & 1u ? x[i] : off;
            }
        };
        mask_rows(s);
        if (first) {
            // a near piece: every query sees at least one of its rows
            float mx = s[0] * cs;
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i] * cs);
            mrun = pair_max(mx);
            first = false;
        }
        // P against the reference maximum as it stands (it only keeps P
        // finite); when a lane's sum passes 2^64 the piece's scores are formed
        // again, m is raised to their maximum and l, dq rescaled
        float bl = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = fexp2(fmaf(s[i], cs, -mrun));
            bl += s[i];
        }
        if (__builtin_amdgcn_ballot_w64(bl > 0x1p64f) != 0) {
            const bool raise = pair_max(bl) > 0x1p64f;   // each query for itself
            read_row(rop, kt, ro);
            s = contract_channels<true>(rop, qo, f32x16{0});
            mask_rows(s);
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[i] * cs);
            mx = pair_max(mx);
            const float mnew = raise ? fmaxf(mrun, mx) : mrun;
            const float corr = fexp2(mrun - mnew);
            lrun *= corr;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                dq0[i] *= corr;
                dq1[i] *= corr;
            }
            mrun = mnew;
            bl = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s[i] = fexp2(fmaf(s[i], cs, -mrun));
                bl += s[i];
            }
        }
        lrun += bl;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] *= dp[i];   // dS
        bf16x8 sb[2];
        pack_b(s, sb);
        contract_tr(kt, to, sb, dq0, dq1);
    };

    const int ntile = nnear + nct;
    for (int t = 0; t < ntile; ++t) {
        const int st = t & 1;
        wait_vm<0>();
        __syncthreads();
        if (t + 1 < ntile) issue(t + 1, st ^ 1);
#pragma unroll 1
        for (int hb = 0; hb < 2; ++hb) {
            const __bf16 *kt = sm.k[st] + hb * 32 * kHeadDim, *vt = sm.v[st] + hb * 32 * kHeadDim;
            int mode = 0;
            uint32_t mw = 0;
            if (t < nnear) {
                if (!piece_used<GEOM>(a, m, 2 * t + hb)) continue;
                if (!TWO_D && t * KT + 32 * hb == m.wdiag) mode = 1;
            } else {
                const int pc = 2 * (t - nnear) + hb;
                if (!m.active || pc < gl.pc0 || pc >= gl.pc0 + gl.npc) continue;
                mw = __builtin_amdgcn_readfirstlane(sm.list.vis[GEOM == GEOM_2DP ? wave >> 1 : 0][pc]);
                if (mw == 0) continue;
                mw >>= 4 * hh;
                mode = 2;
            }
            piece(kt, vt, mode, mw);
        }
    }
    if (!m.active) return;
    const float lsum = pair_sum(lrun);
    if (hh == 0) {
        a.lse[(long long)slice * a.n + qtok] = mrun + __log2f(lsum);
        a.delta[(long long)slice * a.n + qtok] = dd;
    }
    const float f = lsum > 0.f ? a.scale / lsum : 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        dq0[i] *= f;
        dq1[i] *= f;
    }
    store_rows(static_cast<__bf16 *>(a.dq) + (long long)slice * a.n * kHeadDim, dq0, dq1, lane,
               [&](int row) { return wave_token<GEOM>(a, m, m.pos0 + row); });
}

// --------------------------------------------------------- coarse-row pass
// Partial gradients of the coarse rows, dK_bar = tau Q^T dS and dV_bar = dO^T P
// over the queries of one sibling group (group_slots): one wave per (slice,
// group, 32 slots), the slots' rows in registers, the group's queries in
// 32-row chunks through a ring of two private LDS stages: no barrier, no sums
// between waves.  A slot that a block of the group does not list (the level-1
// window's near squares, or a group past the map) is masked for its chunks.
// Sharing one partial row among the siblings is what makes it cheap in 2D: 90
// rows per four cells of a three-level map instead of 4 x 81, 0.38 GB of
// partials instead of 1.36 (2D at 128 slices: 235 us, 104 us in 1D at 96).
struct CoarseSmem {
    __bf16 q[2][32 * kHeadDim];
    __bf16 g[2][32 * kHeadDim];
    __attribute__((aligned(16))) float ld[2][64];   // lse of the chunk's rows, then D
};

template <bool TWO_D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 3))) void bwd_coarse_mfma(BwdArgs a)
{
    __shared__ __attribute__((aligned(16))) CoarseSmem sm;
    const int lane = threadIdx.x, l32 = lane & 31, hh = lane >> 5;
    const int npc = (a.gslot + 31) / 32;
    const unsigned id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int pc = (int)(id % (unsigned)npc);
    const unsigned gid = id / (unsigned)npc;
    const int ls = (int)(gid / (unsigned)a.ngrp), grp = (int)(gid - (unsigned)ls * (unsigned)a.ngrp);
    const int slice = a.slice0 + ls;

    const SiblingGroup sg = sibling_group<TWO_D>(a, grp);
    const int nchunk = sg.ncx * sg.ncy * sg.cpb;

    // this lane's slot: its coarse row and the blocks that list it
    int mask;
    const int row = sibling_slot<TWO_D>(a, sg, a.gslot, pc * 32 + l32, mask);
    RowOp<true> ko, vn;   // the slot's rows (V negated, as in the key pass)
    const long long crow = ((long long)slice * a.R + row) * kHeadDim;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        ko.x[c] = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(a.kbar) + crow + 16 * c + 8 * hh);
        uint4 v = *reinterpret_cast<const uint4 *>(static_cast<const __bf16 *>(a.vbar) + crow + 16 * c + 8 * hh);
        v.x ^= 0x80008000u;
        v.y ^= 0x80008000u;
        v.z ^= 0x80008000u;
        v.w ^= 0x80008000u;
        vn.x[c] = __builtin_bit_cast(bf16x8, v);
    }

    const char *const qg = static_cast<const char *>(a.q) + (long long)slice * a.n * ROWB;
    const char *const gg = static_cast<const char *>(a.dout) + (long long)slice * a.n * ROWB;
    const float *const lg = a.lse + (long long)slice * a.n;
    const float *const dg = a.delta + (long long)slice * a.n;
    const int loff0 = dma_lane_off(lane, 0), loff1 = dma_lane_off(lane, 1);
    auto run_tok = [&](int c, int i8) { return sibling_run<TWO_D>(a, sg, c, i8); };
    auto issue = [&](int c, int st) {   // nine loads
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const long long o = run_tok(c, i) * ROWB + ((i & 1) ? loff1 : loff0);
            dma16(qg + o, lds_u32(sm.q[st]) + i * 1024);
            dma16(gg + o, lds_u32(sm.g[st]) + i * 1024);
        }
        dma4((hh ? dg : lg) + run_tok(c, l32 >> 3) + (l32 & 7), lds_u32(sm.ld[st]));
    };
    issue(0, 0);

    const float cs = a.scale_log2;
    const RowOff ro = row_offsets(l32, hh);
    const TrOff to = tr_offsets(lane);
    f32x16 dk0 = {0}, dk1 = {0}, dv0 = {0}, dv1 = {0};
    for (int c = 0; c < nchunk; ++c) {
        const int st = c & 1;
        if (c + 1 < nchunk) {
            __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // the other stage's reads are done
            issue(c + 1, st ^ 1);
            wait_vm<9>();
        } else {
            wait_vm<0>();
        }
        int bi, bj, bp;
        sibling_block(sg, c, bi, bj, bp);
        const bool on = (mask >> (2 * bi + bj)) & 1;
        RowOp<true> rop;
        read_row(rop, sm.q[st], ro);
        f32x16 s = contract_channels<true>(rop, ko, f32x16{0});   // S: queries x slots
        __builtin_amdgcn_sched_barrier(0);
        read_row(rop, sm.g[st], ro);
        f32x16 dp;
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
            const f32x4 d4 = *reinterpret_cast<const f32x4 *>(&sm.ld[st][32 + 8 * c4 + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) dp[4 * c4 + e] = d4[e];
        }
        dp = contract_channels<true>(rop, vn, dp);                // D - dP
        __builtin_amdgcn_sched_barrier(0);
        f32x16 p;
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
            const f32x4 l4 = *reinterpret_cast<const f32x4 *>(&sm.ld[st][8 * c4 + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[4 * c4 + e] = fexp2(fmaf(s[4 * c4 + e], cs, -l4[e]));
                s[4 * c4 + e] = p[4 * c4 + e] * dp[4 * c4 + e];   // -dS
            }
        }
        bf16x8 pb[2], sb[2];
        pack_b(p, pb);
        pack_b(s, sb);
        if (__builtin_amdgcn_ballot_w64(!on) != 0) {
            // bitwise, so that a masked slot's weights are 0 whatever they were
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const uint32_t keep = on ? 0xffffffffu : 0u;
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                u32x4 x = __builtin_bit_cast(u32x4, pb[hf]), y = __builtin_bit_cast(u32x4, sb[hf]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] &= keep;
                    y[e] &= keep;
                }
                pb[hf] = __builtin_bit_cast(bf16x8, x);
                sb[hf] = __builtin_bit_cast(bf16x8, y);
            }
        }
        contract_tr(sm.g[st], to, pb, dv0, dv1);   // dO^T P
        contract_tr(sm.q[st], to, sb, dk0, dk1);   // -Q^T dS
    }
    const long long base = (((long long)ls * a.ngrp + grp) * a.gslot + pc * 32) * kHeadDim;
    const long long half = (long long)a.pslices * a.ngrp * a.gslot * kHeadDim;
    auto rowptr = [&](float *b) {
        return [&, b](int r) { return pc * 32 + r < a.gslot ? b + r * kHeadDim : static_cast<float *>(nullptr); };
    };
    store_rows_f32(dk0, dk1, -a.scale, lane, rowptr(a.part + base));
    store_rows_f32(dv0, dv1, 1.f, lane, rowptr(a.part + half + base));
}

// dK_bar, dV_bar of every coarse row: one wave per (tensor, slice, row), the
// partial rows of the sibling groups whose lists hold it in a fixed order,
// dealt to eight lane groups (deal_box).  Level 1: the parents next to the
// row's own (3 per axis), slot = place in the parent's window; level l >= 2:
// the sibling groups inside the level-l groups that list it (list inverse).
template <bool TWO_D>
__global__ __launch_bounds__(64) void bwd_group_reduce(BwdArgs a)
{
    constexpr int K = TWO_D ? kSlots2D : kSlots1D, KW = group_window(TWO_D);
    constexpr int NC = TWO_D ? 49 : 7;
    __shared__ int cand_j[NC];
    const long long wg = blockIdx.x;
    const int tid = threadIdx.x;
    const int z = (int)(wg / ((long long)a.pslices * a.R));
    const long long rem = wg - (long long)z * a.pslices * a.R;
    const int ls = (int)(rem / a.R);
    const int crow = (int)(rem - (long long)ls * a.R);
    const int slice = a.slice0 + ls;
    if (z > 1 || slice >= a.nslice) return;
    int e = 0;
    while (e + 1 < a.lv.nlev && a.lv.off[e + 1] <= crow) ++e;
    const int lvl = a.lv.lvl[e], M = a.lv.M[e], My = a.lv.My[e];
    const int g = crow - a.lv.off[e];
    const int u = TWO_D ? g / My : g, v = TWO_D ? g - (g / My) * My : 0;
    const int ngx = (a.nbx + 1) >> 1, ngy = TWO_D ? (a.nby + 1) >> 1 : 1;   // sibling groups per axis
    const int grp = tid >> 3, c8 = (tid & 7) * 8;
    const long long zoff = ((long long)z * a.pslices + ls) * a.ngrp * a.gslot * kHeadDim;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto add = [&](int px, int py, int slot) {
        const long long pr = TWO_D ? (long long)px * ngy + py : px;
        add8(acc, a.part, zoff + (pr * a.gslot + slot) * kHeadDim + c8, a.part_elems);
    };
    if (lvl == 1) {
        const int px0 = (u >> 1) > 0 ? (u >> 1) - 1 : 0, px1 = (u >> 1) + 1 < ngx ? (u >> 1) + 1 : ngx - 1;
        const int py0 = TWO_D && (v >> 1) > 0 ? (v >> 1) - 1 : 0, py1 = TWO_D && (v >> 1) + 1 < ngy ? (v >> 1) + 1 : ngy - 1;
        deal_box<8>(px1 - px0 + 1, py1 - py0 + 1, 1, grp, 0, [&](int dx, int dy, int) {
            const int px = px0 + dx, py = py0 + dy;
            const int au = u - (2 * px - 2), av = v - (2 * py - 2);
            add(px, py, e * KW + (TWO_D ? au * 6 + av : au));
        });
    } else {
        const int span = 1 << (lvl - 2);   // sibling groups per level group and axis
        if (tid < NC) {
            int jj = -1;
            if constexpr (TWO_D) {
                const int qx = u - 3 + tid / 7, qy = v - 3 + tid % 7;
                if (qx >= 0 && qy >= 0 && qx < M && qy < My && qx * span < ngx && qy * span < ngy)
                    jj = list2d_slot_of(qx, qy, u, v);
            } else {
                const int q = g - 3 + tid;
                if (q >= 0 && q < M && q * span < ngx)
                    for (int j = 0; j < K; ++j)
                        if (list1d_entry(2 * q * span, lvl, j, M, a.causal) == g) jj = j;
            }
            cand_j[tid] = jj;
        }
        __syncthreads();
        int t0 = 0;
        for (int c = 0; c < NC; ++c) {
            const int j = cand_j[c];
            if (j < 0) continue;
            const int slot = a.rank * KW + (e - a.rank) * K + j;
            const int px0 = (TWO_D ? u - 3 + c / 7 : g - 3 + c) * span, py0 = TWO_D ? (v - 3 + c % 7) * span : 0;
            const int nx = ngx - px0 < span ? ngx - px0 : span, ny = TWO_D ? (ngy - py0 < span ? ngy - py0 : span) : 1;
            deal_box<8>(nx, ny, 1, grp, t0, [&](int dx, int dy, int) { add(px0 + dx, py0 + dy, slot); });
            t0 += nx * ny;
        }
    }
    store_group_sums(acc, grp, z ? a.dvbar : a.dkbar, ((long long)slice * a.R + crow) * kHeadDim + c8, a.coarse_elems, true);
}

// ------------------------------------------------------------------ key pass
// Gradients of the keys and values: dk, dv from the queries of the near window
// and, through the coarsening, from dK_bar, dV_bar of every coarse set; plus
// the dot products k . dK_bar, v . dV_bar for the weight gradients.
//
// What bounds it: at 1D 65536 x 128, 32 slices, it reads Q, dO, K, V and
// writes dK, dV and the dot products once, 1.7 GB (335 us at the 5.2 TB/s of a
// copy); its matrix products alone would take ~165 us.  Three waves per SIMD
// (168 registers, 36 KB of LDS per workgroup), two LDS stages filled by
// direct loads and one barrier per 64-row tile; D enters as the C operand of
// the dP product.  The coarse-set epilogue takes its operands from L2 as
// ready-made (hi, lo) bf16 pairs, where splitting fp32 rows in place cost
// 320 us of it, and results leave as 64-byte pieces (store_rows) instead of
// 8-byte ones.  Against the register-staged kernel (two barriers per tile, two
// waves per SIMD): 1D 65536 x 128 892 -> 624 us, causal 16384 x 128 (96
// slices) 535 -> 397 us, 128 x 128 map (128 slices) 1172 -> 789 us, blocks of
// 32 (64 slices of 4000) 215 -> 68 us.
struct KeySmem {
    __bf16 q[2][TILEE];   // two stages of 64 query rows
    __bf16 g[2][TILEE];   // and their upstream gradients
    __attribute__((aligned(16))) float lse[2][KT];
    __attribute__((aligned(16))) float dd[2][KT];
    // each wave's base block: per coarse set the element offset of its group's
    // row and its weights' offsets (2D: row and column vector)
    int row[4][kMaxSets], wo[4][kMaxSets], wy[4][kMaxSets];
};

// hi + lo bf16 parts of eight fp32 values
__device__ inline void split8(const float (&x)[8], bf16x8 &h, bf16x8 &l)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        h[j] = static_cast<__bf16>(x[j]);
        l[j] = static_cast<__bf16>(x[j] - static_cast<float>(h[j]));
    }
}

// eight (hi, lo) bf16 pairs, hi in the low half, as two operands
__device__ inline void unpack_pairs(const uint32_t (&x)[8], bf16x8 &h, bf16x8 &l)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 a, b;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a[j] = __builtin_amdgcn_perm(x[2 * j + 1], x[2 * j], 0x05040100u);
        b[j] = __builtin_amdgcn_perm(x[2 * j + 1], x[2 * j], 0x07060302u);
    }
    h = __builtin_bit_cast(bf16x8, a);
    l = __builtin_bit_cast(bf16x8, b);
}

template <int GEOM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void bwd_key_mfma(BwdArgs a)
{
    constexpr bool TWO_D = GEOM != GEOM_1D;
    __shared__ __attribute__((aligned(16))) KeySmem sm;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int gps = (int)row_groups<GEOM>(a);
    const int slice = __builtin_amdgcn_readfirstlane((int)(id / (unsigned)gps));
    const int grp = (int)(id - (unsigned)slice * (unsigned)gps);
    const RowGroup m = row_group<GEOM, true>(a, grp, wave);
    constexpr int lgr = GEOM == GEOM_2DP ? 3 : 4;
    const int kp = m.pos0 + l32;   // position of the lane's key in its block
    {
        const int e = lane < a.lv.nlev ? lane : 0;
        int bcx = m.blk, bcy = 0;
        if constexpr (TWO_D) {
            bcx = m.blk / a.nby;
            bcy = m.blk - bcx * a.nby;
        }
        int row = 0, wo = 0, wy = 0;
        if (a.lv.nlev > 0) {
            // s_l = r 2^(l-1): the block's level-l group is b >> (l-1) per axis
            // and the block's place in it b mod 2^(l-1)
            const int sh = a.lv.lvl[e] - 1, msk = (1 << sh) - 1;
            if constexpr (TWO_D) {
                row = a.lv.off[e] + (bcx >> sh) * a.lv.My[e] + (bcy >> sh);
                wo = a.lv.woff[e] + ((bcx & msk) << lgr);
                wy = a.lv.woff[e] + a.lv.size[e] + ((bcy & msk) << lgr);
            } else {
                row = a.lv.off[e] + (bcx >> sh);
                wo = a.lv.woff[e] + (bcx & msk) * a.r;
            }
        }
        sm.row[wave][lane] = row * kHeadDim;
        sm.wo[wave][lane] = wo;
        sm.wy[wave][lane] = wy;
    }

    const char *const qg = static_cast<const char *>(a.q) + (long long)slice * a.n * ROWB;
    const char *const gg = static_cast<const char *>(a.dout) + (long long)slice * a.n * ROWB;
    const float *const lg = a.lse + (long long)slice * a.n;
    const float *const dg = a.delta + (long long)slice * a.n;
    const int loff = dma_lane_off(lane, wave & 1);

    // Tile t into stage st: wave w loads rows 8 w .. and 8 (w + 4) .. of Q
    // and dO; wave 0 the rows' lse, wave 1 their D
    auto issue = [&](int t, int st) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int i = wave + 4 * jj;
            const long long o = window_run<GEOM>(a, m, 8 * t + i) * ROWB + loff;
            dma16(qg + o, lds_u32(sm.q[st]) + i * 1024);
            dma16(gg + o, lds_u32(sm.g[st]) + i * 1024);
        }
        if (wave < 2) {
            const long long tok = window_run<GEOM>(a, m, 8 * t + (lane >> 3)) + (lane & 7);
            dma4((wave == 0 ? lg : dg) + tok, lds_u32(wave == 0 ? sm.lse[st] : sm.dd[st]));
        }
    };
    issue(0, 0);

    // this lane's key; V enters negated, so that D - dO . v comes out of the
    // matrix cores with D as the C operand
    const long long ktok = m.active ? wave_token<GEOM>(a, m, m.pos0 + l32) : 0;
    const long long krow = ((long long)slice * a.n + ktok) * kHeadDim;
    RowOp<true> ko, vn;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        ko.x[c] = __builtin_bit_cast(bf16x8, ld16(a.k, krow + 16 * c + 8 * hh, 2, a.io_elems));
        uint4 v = ld16(a.v, krow + 16 * c + 8 * hh, 2, a.io_elems);
        v.x ^= 0x80008000u;
        v.y ^= 0x80008000u;
        v.z ^= 0x80008000u;
        v.w ^= 0x80008000u;
        vn.x[c] = __builtin_bit_cast(bf16x8, v);
    }
    const float cs = a.scale_log2;
    const RowOff ro = row_offsets(l32, hh);
    const TrOff to = tr_offsets(lane);

    f32x16 dk0 = {0}, dk1 = {0}, dv0 = {0}, dv1 = {0};
    const int ntile = (m.npiece + 1) / 2;
    for (int t = 0; t < ntile; ++t) {
        const int st = t & 1;
        wait_vm<0>();
        __syncthreads();
        if (t + 1 < ntile) issue(t + 1, st ^ 1);
#pragma unroll 1
        for (int qb = 0; qb < 2; ++qb) {
            if (!piece_used<GEOM>(a, m, 2 * t + qb)) continue;
            const __bf16 *qt = sm.q[st] + qb * 32 * kHeadDim, *gt = sm.g[st] + qb * 32 * kHeadDim;
            // (the fences keep the two row operands from being live at once:
            // the next one's reads run under the previous one's products)
            RowOp<true> rop;
            read_row(rop, qt, ro);
            f32x16 s = contract_channels<true>(rop, ko, f32x16{0});   // S: queries x keys
            __builtin_amdgcn_sched_barrier(0);
            read_row(rop, gt, ro);
            f32x16 dp;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 d4 = *reinterpret_cast<const f32x4 *>(&sm.dd[st][qb * 32 + 8 * c + 4 * hh]);
#pragma unroll
                for (int e = 0; e < 4; ++e) dp[4 * c + e] = d4[e];
            }
            dp = contract_channels<true>(rop, vn, dp);                // D - dP
            __builtin_amdgcn_sched_barrier(0);
            f32x16 p;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 l4 = *reinterpret_cast<const f32x4 *>(&sm.lse[st][qb * 32 + 8 * c + 4 * hh]);
#pragma unroll
                for (int e = 0; e < 4; ++e) p[4 * c + e] = fexp2(fmaf(s[4 * c + e], cs, -l4[e]));
            }
            if constexpr (!TWO_D)
                if (t * KT + 32 * qb == m.wdiag) {   // causal: the wave's own rows, query >= key
#pragma unroll
                    for (int i = 0; i < 16; ++i) p[i] = acc_row(i, hh) >= l32 ? p[i] : 0.f;
                }
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = p[i] * dp[i];   // -dS
            bf16x8 pb[2], sb[2];
            pack_b(p, pb);
            contract_tr(gt, to, pb, dv0, dv1);   // dO^T P
            pack_b(s, sb);
            contract_tr(qt, to, sb, dk0, dk1);   // -Q^T dS
        }
    }
    if (!m.active) return;
    const float nsc = -a.scale;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        dk0[i] *= nsc;
        dk1[i] *= nsc;
    }

    // coarse sets, 16 at a time (k slots = sets; every key of the wave lies in
    // the same group of every set):
    //   dk^T += dK_bar^T W^k, dv^T += dV_bar^T W^v (rows channels, columns
    //   keys) and the dot products k . dK_bar, v . dV_bar (rows sets, columns
    //   keys), with dK_bar, dV_bar and the weights as a bf16 high part and the
    //   bf16 rounding of the rest (hi*hi + lo*hi + hi*lo, error ~2^-17 of each
    //   product; k and v are exact).  The reduction leaves dK_bar, dV_bar as
    //   such pairs; the operands come straight from L2: no LDS, no barrier.
    const long long rbase = (long long)slice * a.R * kHeadDim;
    const long long wbase = a.w_stride ? (long long)(slice % a.heads) * a.wlen : 0;
    const long long dbase = (long long)slice * a.lv.nlev * a.n + ktok;
    auto add_sets = [&](int e0, const uint32_t *src, const float *wsrc, const RowOp<true> &op, uint32_t flip, float *dst,
                        f32x16 &d0, f32x16 &d1) {
        {
            // B operand: the weights of sets e0 + 8 hh .. + 7 for this key; A
            // operands: channel 32 db + l32 of those sets' rows
            float wt[8];
            uint32_t x0[8], x1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int e = e0 + 8 * hh + j;   // (sets past the last one: row 0, weight 0)
                if constexpr (TWO_D)
                    wt[j] = wsrc[sm.wo[wave][e] + (kp >> lgr)] * wsrc[sm.wy[wave][e] + (kp & ((1 << lgr) - 1))];
                else
                    wt[j] = wsrc[sm.wo[wave][e] + kp];
                wt[j] = e < a.lv.nlev ? wt[j] : 0.f;
                x0[j] = src[sm.row[wave][e] + l32];
                x1[j] = src[sm.row[wave][e] + 32 + l32];
            }
            bf16x8 wh, wl, h, l;
            split8(wt, wh, wl);
            unpack_pairs(x0, h, l);
            d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, wh, d0, 0, 0, 0);
            d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l, wh, d0, 0, 0, 0);
            d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, wl, d0, 0, 0, 0);
            unpack_pairs(x1, h, l);
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, wh, d1, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l, wh, d1, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, wl, d1, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // dots: A rows are the chunk's 16 sets (lanes 16 .. 31 repeat them)
        const uint32_t *const rm = src + sm.row[wave][e0 + (l32 & 15)] + 8 * hh;
        f32x16 td = {0};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint4 p0 = *reinterpret_cast<const uint4 *>(rm + 16 * c);
            const uint4 p1 = *reinterpret_cast<const uint4 *>(rm + 16 * c + 4);
            const uint32_t x[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
            bf16x8 h, l;
            unpack_pairs(x, h, l);
            td = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h, op.x[c], td, 0, 0, 0);
            td = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l, op.x[c], td, 0, 0, 0);
        }
        float *dp = dst + (long long)(e0 + 4 * hh) * a.n;   // rows 0 .. 15: this chunk's sets
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (e0 + acc_row(i, hh) < a.lv.nlev) *dp = __uint_as_float(__float_as_uint(td[i]) ^ flip);
            dp += (i == 3 ? 5 : 1) * a.n;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll 1
    for (int ec = 0; ec < a.lv.nlev; ec += 16) {
        int e0 = ec;
        asm volatile("" : "+s"(e0));   // keeps the chunk's addresses out of registers until here
        add_sets(e0, reinterpret_cast<const uint32_t *>(a.dkbar) + rbase, a.wk + wbase, ko, 0u, a.dotk + dbase, dk0, dk1);
        add_sets(e0, reinterpret_cast<const uint32_t *>(a.dvbar) + rbase, a.wv + wbase, vn, 0x80000000u, a.dotv + dbase,
                 dv0, dv1);
    }
    store_rows(static_cast<__bf16 *>(a.dk) + (long long)slice * a.n * kHeadDim, dk0, dk1, lane,
               [&](int row) { return wave_token<GEOM>(a, m, m.pos0 + row); });
    store_rows(static_cast<__bf16 *>(a.dv) + (long long)slice * a.n * kHeadDim, dv0, dv1, lane,
               [&](int row) { return wave_token<GEOM>(a, m, m.pos0 + row); });
}

template <int GEOM>
hipError_t launch_key(const BwdArgs &a, hipStream_t st)
{
    const long long groups = (long long)a.nslice * row_groups<GEOM>(a);
    if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((bwd_key_mfma<GEOM>), dim3((unsigned)groups), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int GEOM>
hipError_t launch_query(const BwdArgs &a, hipStream_t st)
{
    constexpr bool TWO_D = GEOM != GEOM_1D;
    const long long groups = (long long)a.nslice * row_groups<GEOM>(a);
    if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
    if (!group_lists_fit<GEOM>(a)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((bwd_query_mfma<GEOM>), dim3((unsigned)groups), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.lv.nlev == 0) return e;
    // the coarse rows' gradients, pslices slices at a time
    if (a.pslices <= 0 || 2LL * a.pslices * a.ngrp * a.gslot * kHeadDim > a.part_elems) return hipErrorInvalidValue;
    for (int s0 = 0; s0 < a.nslice; s0 += a.pslices) {
        BwdArgs b = a;
        b.slice0 = s0;
        const int cnt = a.nslice - s0 < a.pslices ? a.nslice - s0 : a.pslices;
        const long long units = (long long)cnt * a.ngrp * ((a.gslot + 31) / 32), rows = 2LL * a.pslices * a.R;
        if (units > 0x7fffffffLL || rows > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL((bwd_coarse_mfma<TWO_D>), dim3((unsigned)units), dim3(64), 0, st, b);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL((bwd_group_reduce<TWO_D>), dim3((unsigned)rows), dim3(64), 0, st, b);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_bwd_query(const BwdArgs &a, bool two_d, hipStream_t st)
{
    if (!backward_streams(a.n, a.R, a.r, two_d)) return hipErrorInvalidValue;
    if (!two_d) return launch_query<GEOM_1D>(a, st);
    return a.r == 8 ? launch_query<GEOM_2DP>(a, st) : launch_query<GEOM_2D>(a, st);
}

hipError_t launch_bwd_key(const BwdArgs &a, bool two_d, hipStream_t st)
{
    if (!backward_streams(a.n, a.R, a.r, two_d)) return hipErrorInvalidValue;
    if (!two_d) return launch_key<GEOM_1D>(a, st);
    return a.r == 8 ? launch_key<GEOM_2DP>(a, st) : launch_key<GEOM_2D>(a, st);
}

}  // namespace fma_dev
