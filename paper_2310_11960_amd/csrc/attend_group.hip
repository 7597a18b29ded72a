// attend_group.hip -- fused multilevel FMA attention for bf16 on groups of 128
// queries (row_groups.hpp): any block of a multiple of 32 tokens, 2D cells of
// 8 x 8 and 16 x 16, head dims 32, 64 and 128, either normalisation
// (attend_route.hpp tells where it is taken).
//
// What bounds it: at 1D 65536 x 128, 32 slices, its loads and stores alone take
// 181 us (1.08 GB at 6 TB/s) and its arithmetic alone 250-295 us (matrix and
// vector instructions of a 32 x 32 piece, 256 + ~350 cycles); two, three or
// four waves per SIMD, and two pieces at a time, measure the same.  Between
// that and the kernel's time lies the start of every group, ~5 us of set
// tables, list table, queries and first tile before 13.5 us of loop, which only
// the CU's other workgroups hide: the dense reference runs the same arithmetic
// per piece at 856 TFLOP/s (16 384 keys a query), this kernel a 128 x 128 map
// at 573.
//
// Four waves of 32 queries share the group's near window and list rows, which
// stream through two LDS stages of at most 8 KB per tensor (32 rows at d =
// 128, else 64) by direct-to-LDS loads, one barrier per tile; a wave takes the
// 32-row pieces of its own block's window and list.  Per piece:
//   S^T = K Q^T (ds_read_b128 rows, Q in registers), P = exp2(c s - m), l the
//   fp32 sum of P (SQ: of the bf16 P), O^T += V^T P^T (transposing LDS reads).
//   m is the running maximum, or (SQ) the first piece's, raised only when a
//   lane's weights would pass 2^64.
// Each row's 16-byte chunk c sits at chunk c ^ swzd(row).
#include "attend_route.hpp"
#include "level_weights.hpp"

namespace fma_dev {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// The swizzle keeps both the row reads of a 32x32 operand (lane = row) and the
// transposing reads (four rows of two chunks per 16 lanes) on distinct banks;
// rows are 64, 128 or 256 bytes.
template <int D>
__device__ inline int swzd(int row)
{
    const int s64 = (2 * (row & 3)) ^ ((row >> 2) & 1) ^ (2 * ((row >> 3) & 1));
    if constexpr (D == 32) return (2 * ((row >> 1) & 1)) ^ ((row >> 2) & 1);
    else if constexpr (D == 64) return s64;
    else return s64 ^ (8 * (row & 1));
}

template <int D>
constexpr int kTileRows = D == 128 ? 32 : 64;

template <int D>
struct GroupSmem {
    __bf16 k[2][kTileRows<D> * D];
    __bf16 v[2][kTileRows<D> * D];
    ListSmem list;
    SetTab st;
};

__device__ inline float gexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline int grow(int i, int hh) { return 8 * (i >> 2) + 4 * hh + (i & 3); }   // accumulator row

// PL: printed per-level normalisation (levels inside a 32-slot piece).
// SQ (scaled queries): c Q rounded to bf16, no running maximum and l from the
// bf16 weights, as attend_mfma.hip has them, for the block sizes both kernels
// take (d = 64, blocks of 64 and more).  The two still differ by rounding: that
// kernel subtracts m inside the matrix product and checks 16 rows at a time.
// The others keep the fp32 scale, the running maximum and the fp32 row sum of
// attend.hip; under the running maximum a dominating source's weight is exactly
// 1: without it the error against float64 was 4 % larger (2.24e-3 against
// 2.14e-3), for 122 instead of 154 us at d = 128.
template <int D, int GEOM, bool PL, bool SQ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : PL || !SQ ? 3 : 4)))
void attend_group_kernel(AttnArgs a)
{
    constexpr int TR = kTileRows<D>, PPT = TR / 32, CPR = D / 8, RI = 64 / CPR, NLD = TR / RI;   // NLD loads per tensor
    constexpr int NC = D / 16, ND = D / 32, RB = 2 * D;
    __shared__ __attribute__((aligned(16))) GroupSmem<D> sm;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int gps = (int)row_groups<GEOM>(a);
    const int slice = __builtin_amdgcn_readfirstlane((int)(id / (unsigned)gps));
    const int grp = (int)(id - (unsigned)slice * (unsigned)gps);
    const RowGroup m = row_group<GEOM, false>(a, grp, wave);
    load_sets(sm.st, a, tid);

    const char *const kg = static_cast<const char *>(a.k) + (long long)slice * a.n * RB;
    const char *const vg = static_cast<const char *>(a.v) + (long long)slice * a.n * RB;
    const char *const kb = static_cast<const char *>(a.kbar) + (long long)slice * a.R * RB;
    const char *const vb = static_cast<const char *>(a.vbar) + (long long)slice * a.R * RB;
    const GroupLists gl = group_lists<GEOM, PL>(a, m, grp, wave);
    const int nnear = (m.npiece + PPT - 1) / PPT, nct = (gl.npiece + PPT - 1) / PPT;   // near and coarse tiles
    const int lr = lane / CPR, lp = lane % CPR;

    // Tile t into stage st: NLD loads per tensor, wave w takes w, w + 4, .. of both
    auto issue = [&](int t, int st) __attribute__((always_inline)) {
        const bool co = t >= nnear;
        TileCell cell = {0, 0};
        if (!co) cell = tile_cell<GEOM, TR>(a, m, t);
#pragma unroll
        for (int jj = 0; jj < NLD / 4; ++jj) {
            const int i = wave + 4 * jj, row = i * RI + lr;
            const int ch = 16 * (lp ^ swzd<D>(row));
            const uint32_t kd = lds_u32(sm.k[st]) + i * 1024, vd = lds_u32(sm.v[st]) + i * 1024;
            if (co) {
                const int x = sm.list.crow[(t - nnear) * TR + row];   // (a piece without rows, which no wave takes: row 0)
                const long long r = (long long)(x < 0 ? 0 : x) * RB + ch;
                dma16(kb + r, kd);
                dma16(vb + r, vd);
            } else {
                const long long r = tile_token<GEOM, TR>(a, m, cell, t, row);
                dma16(kg + r * RB + ch, kd);
                dma16(vg + r * RB + ch, vd);
            }
        }
    };
    issue(0, 0);

    // this lane's query (waves without rows repeat token 0 and store nothing)
    const long long qtok = m.active ? wave_token<GEOM>(a, m, m.pos0 + l32) : 0;
    bf16x8 qo[NC];
    {
        const __bf16 *qp = static_cast<const __bf16 *>(a.q) + ((long long)slice * a.n + qtok) * D + 8 * hh;
#pragma unroll
        for (int c = 0; c < NC; ++c) qo[c] = *reinterpret_cast<const bf16x8 *>(qp + 16 * c);
    }
    __syncthreads();   // the set tables
    build_lists<GEOM, PL>(a, m, gl, grp, sm.st, wave, lane, sm.list);

    // operand offsets (elements) in a tile: chunk 2 c + hh of row l32 is
    // koff ^ 16 c; the transposing reads of channels 32 db .. and rows 0 .. 15
    // are voff[h] ^ 32 db
    const int koff = l32 * D + 8 * (hh ^ swzd<D>(l32));
    int voff[2];
    {
        const int gq = lane >> 4, s4 = lane & 15, j = s4 >> 2, q = s4 & 3;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = 8 * h + 4 * (gq >> 1) + j;
            voff[h] = row * D + 8 * ((2 * (gq & 1) + (q >> 1)) ^ swzd<D>(row)) + 4 * (q & 1);
        }
    }

    const float cs = a.scale_log2;
    // a masked score: -inf once scaled (the scale may be negative)
    const float off = !SQ && cs < 0.f ? INFINITY : -INFINITY;
    if constexpr (SQ) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) qo[c][e] = static_cast<__bf16>(static_cast<float>(qo[c][e]) * cs);
    }
    f32x16 o[ND];
#pragma unroll
    for (int db = 0; db < ND; ++db) o[db] = f32x16{0};
    float mrun = 0.f, lrun = 0.f;
    bool first = true;
    auto scores = [&](const __bf16 *kt) __attribute__((always_inline)) {
        f32x16 s = {0};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // (d = 128: four row chunks in registers at a time)
            if (D == 128 && c == NC / 2) __builtin_amdgcn_sched_barrier(0);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(kt + (koff ^ (16 * c))), qo[c],
                                                        s, 0, 0, 0);
        }
        return s;
    };
    // O^T += V^T P^T, P as packed bf16 pairs (element 2 x, 2 x + 1 of the piece's
    // accumulator in w[x])
    auto pv = [&](const uint32_t (&w)[8], const __bf16 *vt) __attribute__((always_inline)) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 pw = {w[4 * hf], w[4 * hf + 1], w[4 * hf + 2], w[4 * hf + 3]};
            const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
            const __bf16 *t16 = vt + 16 * hf * D;
#pragma unroll
            for (int db = 0; db < ND; ++db) {
                if (D == 128 && db == ND / 2) __builtin_amdgcn_sched_barrier(0);
                const s16x4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + (voff[0] ^ (32 * db))));
                const s16x4 r2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t16 + (voff[1] ^ (32 * db))));
                const s16x8 av = {r1[0], r1[1], r1[2], r1[3], r2[0], r2[1], r2[2], r2[3]};
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), pb, o[db], 0, 0, 0);
            }
        }
    };
    // one 32-row piece; mode 0: every row visible, 1: causal diagonal (row <=
    // query), 2: rows whose bit 8 (i >> 2) + (i & 3) of mw is set
    auto piece = [&](const __bf16 *kt, const __bf16 *vt, int mode, uint32_t mw) __attribute__((always_inline)) {
        f32x16 s = scores(kt);
        auto mask_rows = [&](f32x16 &x) {
            if (mode == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = grow(i, hh) <= l32 ? x[i] : off;
            } else if (mode == 2) {
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = (mw >> (8 * (i >> 2) + (i & 3))) & 1u ? x[i] : off;
            }
        };
        mask_rows(s);
        // the weights against m as it stands (it only keeps them finite) and
        // their sum: of the fp32 weights, or (SQ) of their bf16 roundings
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
        uint32_t w[8];
        auto weights = [&]() __attribute__((always_inline)) {
            float bl = 0.f;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const float x0 = SQ ? s[2 * x] - mrun : fmaf(s[2 * x], cs, -mrun);
                const float x1 = SQ ? s[2 * x + 1] - mrun : fmaf(s[2 * x + 1], cs, -mrun);
                const float p0 = gexp2(x0), p1 = gexp2(x1);
                w[x] = pack_bf16(p0, p1);
                if constexpr (SQ)
                    bl = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[x]), ones, bl, false);
                else
                    bl += p0 + p1;
            }
            return bl;
        };
        auto max16 = [&]() __attribute__((always_inline)) {   // maximum of the query's scores, log2 units
            const float f = SQ ? 1.f : cs;
            float mx = s[0] * f;
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i] * f);
            return pair_max(mx);
        };
        // raise m to the piece's maximum and rescale l, O where `up` holds --
        // each query for itself (the others keep m and scale by exp2(0) = 1)
        auto raise = [&](float mx, bool up) __attribute__((always_inline)) {
            const float mnew = up ? fmaxf(mrun, mx) : mrun;
            const float corr = gexp2(mrun - mnew);
            mrun = mnew;
            lrun *= corr;
#pragma unroll
            for (int db = 0; db < ND; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= corr;
        };
        if (first) {
            // a near piece: every query sees at least one of its rows
            mrun = max16();
            first = false;
        } else if constexpr (!SQ) {
            // the running maximum, so that a dominating source's weight is 1
            // exactly and bf16 rounds nothing of it
            const float mx = max16();
            if (__builtin_amdgcn_ballot_w64(mx > mrun) != 0) raise(mx, true);
        }
        float bl = weights();
        if constexpr (SQ) {
            // m as it stands; only where a lane's weights pass 2^64 (a score
            // more than ~60 above m) it is raised and the weights redone
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(bl > 0x1p64f) != 0, 0)) {
                raise(max16(), pair_max(bl) > 0x1p64f);
                bl = weights();
            }
        }
        lrun += bl;
        pv(w, vt);
    };

    const int ntile = nnear + nct;
    float lnear = 0.f;
    for (int t = 0; t < ntile; ++t) {
        const int st = t & 1;
        wait_vm<0>();
        __syncthreads();
        if (t + 1 < ntile) issue(t + 1, st ^ 1);
#pragma unroll 1
        for (int hb = 0; hb < PPT; ++hb) {
            const __bf16 *kt = sm.k[st] + hb * 32 * D, *vt = sm.v[st] + hb * 32 * D;
            int mode = 0;
            uint32_t mw = 0;
            if (t < nnear) {
                const int p = PPT * t + hb;
                if (p >= m.npiece || !piece_used<GEOM>(a, m, p)) continue;
                if (GEOM == GEOM_1D && 32 * p == m.wdiag) mode = 1;
            } else {
                const int pc = PPT * (t - nnear) + hb;
                if (!m.active || pc < gl.pc0 || pc >= gl.pc0 + gl.npc) continue;
                if (PL && pc == gl.pc0) lnear = pair_sum(lrun);   // the near field's row sum, final by now
                mw = __builtin_amdgcn_readfirstlane(sm.list.vis[GEOM == GEOM_2DP && !PL ? wave >> 1 : 0][pc]);
                if (mw == 0) continue;
                mw >>= 4 * hh;
                mode = 2;
                if constexpr (PL) {
                    // every level of the piece normalised on its own and
                    // weighted by the near field's row sum
                    f32x16 s = scores(kt);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        s[i] = (mw >> (8 * (i >> 2) + (i & 3))) & 1u ? s[i] * (SQ ? 1.f : cs) : -INFINITY;
                    level_weights(s, lnear, a.slot_group);
                    uint32_t w[8];
#pragma unroll
                    for (int x = 0; x < 8; ++x) w[x] = pack_bf16(s[2 * x], s[2 * x + 1]);
                    pv(w, vt);
                    continue;
                }
            }
            piece(kt, vt, mode, mw);
        }
    }
    if (!m.active) return;
    const float inv = 1.0f / pair_sum(lrun);
    const int l16 = lane & 15;
    __bf16 *const ob = static_cast<__bf16 *>(a.out) + (long long)slice * a.n * D + 8 * store_chunk(lane);
    __bf16 *const r0 = ob + wave_token<GEOM>(a, m, m.pos0 + l16) * D;
    __bf16 *const r1 = ob + wave_token<GEOM>(a, m, m.pos0 + 16 + l16) * D;
#pragma unroll
    for (int db = 0; db < ND; ++db) store_rows32(o[db], inv, r0 + 32 * db, r1 + 32 * db);
}

template <int D, int GEOM>
hipError_t launch_d(const AttnArgs &a, hipStream_t st)
{
    const long long groups = (long long)a.nslice * row_groups<GEOM>(a);
    if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool pl = a.norm_level && a.nslot > 0;
    if constexpr (D == kHeadDim) {
        if (GEOM != GEOM_1D || a.r >= 64) {
            if (pl)
                hipLaunchKernelGGL((attend_group_kernel<D, GEOM, true, true>), dim3((unsigned)groups), dim3(256), 0, st, a);
            else
                hipLaunchKernelGGL((attend_group_kernel<D, GEOM, false, true>), dim3((unsigned)groups), dim3(256), 0, st, a);
            return hipGetLastError();
        }
    }
    if constexpr (D != kHeadDim || GEOM == GEOM_1D) {
        if (pl)
            hipLaunchKernelGGL((attend_group_kernel<D, GEOM, true, false>), dim3((unsigned)groups), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((attend_group_kernel<D, GEOM, false, false>), dim3((unsigned)groups), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

template <int D>
hipError_t launch_g(const AttnArgs &a, bool two_d, hipStream_t st)
{
    if (!two_d) return launch_d<D, GEOM_1D>(a, st);
    return a.r == 8 ? launch_d<D, GEOM_2DP>(a, st) : launch_d<D, GEOM_2D>(a, st);
}

}  // namespace

bool group_attends(const AttnArgs &a, bool two_d)
{
    const unsigned k = attend_kernels(a, two_d);
    return k == ATTEND_GROUPS || (k == (ATTEND_GROUPS | ATTEND_STREAM) && groups_win(a, compute_units()));
}

hipError_t launch_attend_group(const AttnArgs &a, bool two_d, hipStream_t st)
{
    if (a.nslice == 0 || a.tiles_per_slice == 0) return hipSuccess;
    if (!group_fits(a, two_d)) return hipErrorInvalidValue;
    switch (a.head_dim) {
    case 32: return launch_g<32>(a, two_d, st);
    case 64: return launch_g<64>(a, two_d, st);
    case 128: return launch_g<128>(a, two_d, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fma_dev
