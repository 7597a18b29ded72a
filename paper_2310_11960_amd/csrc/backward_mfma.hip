// backward_mfma.hip -- the bf16 backward on streams of direct-to-LDS tiles
// (see backward.hip for the method and bwd_tiles.hpp for the groups of rows
// and their windows).
#include "bwd_tiles.hpp"

namespace fma_dev {

namespace {

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
    const int slice = (int)(id / (unsigned)gps);
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
            const long long o = tile_run<GEOM>(a, m, t, i) * ROWB + loff;
            dma16(qg + o, lds_u32(sm.q[st]) + i * 1024);
            dma16(gg + o, lds_u32(sm.g[st]) + i * 1024);
        }
        if (wave < 2) {
            const long long tok = tile_run<GEOM>(a, m, t, lane >> 3) + (lane & 7);
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
    for (int t = 0; t < m.ntile; ++t) {
        const int st = t & 1;
        wait_vm<0>();
        __syncthreads();
        if (t + 1 < m.ntile) issue(t + 1, st ^ 1);
#pragma unroll 1
        for (int qb = 0; qb < 2; ++qb) {
            if (!tile_used<GEOM>(m, t, qb)) continue;
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

}  // namespace

// Blocks that the 128-row groups cut into whole 32-row chunks: every 1D block
// of a multiple of 32 and 2D cells of 8 x 8 and 16 x 16.  Blocks of 16 and
// 4 x 4 cells (half a chunk) stay on the register-staged kernels, which pack
// them with idle lanes.
bool bwd_streams(const BwdArgs &a, bool two_d)
{
    // 32-bit tokens and coarse-row element offsets
    if (a.n > 0x7fffffffLL - 4096 || (long long)a.R * kHeadDim > 0x7fffffffLL) return false;
    return two_d ? a.r == 8 || a.r == 16 : a.r % 32 == 0;
}

hipError_t launch_bwd_key(const BwdArgs &a, bool two_d, hipStream_t st)
{
    if (!bwd_streams(a, two_d)) return hipErrorInvalidValue;
    if (!two_d) return launch_key<GEOM_1D>(a, st);
    return a.r == 8 ? launch_key<GEOM_2DP>(a, st) : launch_key<GEOM_2D>(a, st);
}

}  // namespace fma_dev
