// Reorder-gather fused with the block x bitwidth cost table, the kernel and its launch: see fused.hip, which holds the instances for 64-
// and 128-column blocks, and fused_copies.hip, which holds those for 32- and 256-column blocks.
#pragma once

#include <string.h>

#include <vector>

#include "cost_core.hpp"
#include "pack_core.hpp"
#include "surrogate_core.hpp"
#include "sbits_device.hpp"
#include "sbits_internal.hpp"

void sbits_fill_grid_consts(const int32_t *bits, int K, sbits::GridConsts *gc);

namespace sbits {

constexpr int FU_OPU = 16;                          // octets per workgroup at most (128 output rows); fewer for small classes
constexpr int FU_MAX_COLS = 16384;                  // widest row the cost kernel stages (2048 chunks: bf16 + fp32 row in LDS)
constexpr int FU_PACK_MAX_COLS = 32768;             // widest row the packing kernel stages (bf16 row only)

__device__ __forceinline__ int funi(int v) { return __builtin_amdgcn_readfirstlane(v); }

typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) float lds_f32;

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every global
// load in flight, which would expose the latency of the rows being prefetched into registers.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- rows into LDS without passing through registers -------------------------------------
// A wave-wide direct load (16 bytes per lane) writes one contiguous KiB of LDS, "a piece".  The
// RS source rows of a step are laid out piece by piece with the rows interleaved:
//   weights        piece p (columns 512p ..) of row r at  Wb + (p * RS + r) * 1024
//   sensitivities  piece p (columns 256p ..) of row r at  Sb + (p * RS + r) * 1024,  Sb = Wb + nW * RS * 1024
// so one address register per element serves every row of the step (row r = offset r * 1024 of the
// LDS instruction).  The loads carry the non-temporal hint: without it the same loop streams 12 %
// slower.  Lanes past a row's end repeat its last 16 bytes (into the padding of the last piece).
__device__ __forceinline__ void load_row_pieces(const char *wrow, const char *srow, int nW, int nS, uint32_t wbytes,
                                                uint32_t sbytes, uint32_t Wb, uint32_t Sb, int RSr, int rs, int wave,
                                                int nwv, int lane, bool do_w = true, bool do_s = true)
{
    const uint32_t l16 = (uint32_t)lane * 16u;
    for (int p = wave; do_w && p < nW; p += nwv) {
        const uint32_t off = min((uint32_t)p * 1024u + l16, wbytes - 16u);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(wrow + off),
                                         (__attribute__((address_space(3))) void *)(Wb + (uint32_t)(p * RSr + rs) * 1024u),
                                         16, 0, 2);
    }
    for (int p = wave; do_s && p < nS; p += nwv) {
        const uint32_t off = min((uint32_t)p * 1024u + l16, sbytes - 16u);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(srow + off),
                                         (__attribute__((address_space(3))) void *)(Sb + (uint32_t)(p * RSr + rs) * 1024u),
                                         16, 0, 2);
    }
}

// bytes of LDS a step needs: rs rows of cols bf16 weights and (with_s) fp32 sensitivities, in whole pieces
static inline size_t staged_step_bytes(int64_t cols, int rs, bool with_s)
{
    const size_t nW = (size_t)(2 * cols + 1023) / 1024, nS = with_s ? (size_t)(4 * cols + 1023) / 1024 : 0;
    return (nW + nS) * (size_t)rs * 1024;
}

// One element out of the staged rows: the weight (bf16) is loaded into the upper half of a register
// (d16_hi).  On a GPU whose memories run with error correction (the target id says "sramecc+"; every
// MI355X does) such a load writes the whole register, zeros below: the register then holds the weight
// as a float, no conversion instruction needed.  (Without error correction the lower half would keep
// its old contents: the library refuses the one-pass route on such a device, and the packing kernel masks it.)  The compiler does not
// see these loads' completion: lds_gather_wait() below stands between them and the first use.
template <int OFF>
__device__ __forceinline__ void lds_w_hi(float &w, uint32_t addr)
{
    asm volatile("ds_read_u16_d16_hi %0, %1 offset:%2" : "=v"(w) : "v"(addr), "n"(OFF) : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_s(float &s, uint32_t addr)
{
    asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(s) : "v"(addr), "n"(OFF) : "memory");
}
__device__ __forceinline__ void lds_gather_wait(float (&w)[8])
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7])
                 :: "memory");
}
__device__ __forceinline__ void lds_gather_wait(float (&w)[8], float (&s)[8])
{
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7]),
                   "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "+v"(s[4]), "+v"(s[5]), "+v"(s[6]), "+v"(s[7])
                 :: "memory");
}

// Launched with T = the smallest multiple of 64 threads whose CPL chunks per lane cover a row
// (T <= TMAX), so that rows whose chunk count is no power of two leave no lanes idle.
// SUR = false: the block x bitwidth cost table (K candidates per block; with Z0 the first of them is
//              "0 bits", the pruned block, and gc holds the other K - 1 grids).
// SUR = true : the dynamic-sensitivity surrogates (K = 2 sums per block, at the block's current
//              level[]; the "sensitivity" input is the gradient; gc holds every candidate).
// Steps: RS rows each.  Per step: wait for the rows (this wave's loads, then everybody's: barrier),
// pick the lane's elements out of LDS, barrier (the buffer is free), request the next step's rows,
// score.  U = 8 / RS (RS = 2) or 2 (RS = 1) steps are unrolled so that the rows' positions in the
// octet's adjacent-pair tree are compile-time constants.
// Who talks to global memory: a wave that waits for its row loads (vmcnt 0) would also wait for any
// store it has issued, and a store's acknowledgement under this read load takes far longer than a
// load (the octet sums, 16 bytes per block, cost 12 % of the kernel's time that way).  So all waves
// but the last request rows and never store; the octet sums go through a small LDS table and the
// last wave, which requests nothing and never waits for vector memory, writes them out one step later.
// (A workgroup of a single wave does both.)
// SLATE (one row per step, cost table only): the sensitivities are read out of LDS while the first half
// of the arithmetic runs.  Order of a step: weights out of LDS, barrier, request the next row's weights;
// sensitivities requested from LDS (ordinary loads: the compiler places the wait at their first use),
// minimum / range / divisions / x meanwhile; barrier, request the next row's sensitivities; candidates.
// With one workgroup per CU (rows of 8192 elements and more) nobody else would fill the time the LDS
// needs for the gather.
// WPIPE (a refinement of SLATE; the parameter is the distance of the buffers in bytes, 0 = off): two buffers for
// the row of weights, a fixed distance apart (an immediate offset of the LDS reads; at least a row of weights).  The weights of row r + 1 are in LDS a step early, and a lane picks its elements of them out of
// LDS while it runs the second half of row r's arithmetic: no phase of a step is LDS reads alone, and a step
// has two barriers instead of three.
template <int LPG, int K, int CPL, int RS, int TMAX, int MINW, bool SUR, bool Z0, bool SLATE = false, int WPIPE = 0>
__global__ __launch_bounds__(TMAX, MINW)
void gather_cost_kernel(const MatDesc *__restrict__ descs, const int *__restrict__ members,
                        const int *__restrict__ wg_start, int n_members,
                        const int32_t *__restrict__ row_perm, const int32_t *__restrict__ col_perm, int m,
                        uint16_t *__restrict__ w_re_all, float *__restrict__ s_re_all, float *__restrict__ part, GridConsts gc,
                        const uint8_t *__restrict__ level, int kstride, int koff, int opu)
{
    // kstride, koff: the K sums of an octet go to part[..][koff .. koff + K) of kstride values (a launch
    // may cover a subset of the candidates)
    static_assert(!SUR || (K == 2 && !Z0), "two sums per block");
    static_assert(RS == 1 || RS == 2, "rows per step");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int rowsrc[FU_OPU * 8];
    constexpr int NIT = RS * CPL;                    // rows x chunks scored per step
    using DP = DivPlan<LPG, K - Z0>;
    constexpr int NG = NIT > 2 ? 2 : NIT;            // items scored together
    constexpr int NI = SUR ? NG : (DP::RP < NG ? DP::RP : NG);   // of which NI share a round of divisions
    constexpr int U = RS == 2 ? 4 : 2;               // steps unrolled: B = U * RS rows with static tree positions
    constexpr int B = U * RS;
    constexpr bool SDER = RS == 1 && CPL >= 2;       // sensitivity address derived from the weight's (saves registers)
    static_assert(NIT % NG == 0 && NG % NI == 0, "step shape");
    static_assert(!SLATE || (RS == 1 && !SUR && SDER && NIT == NG), "late sensitivities: one row, one group of items");
    static_assert(!WPIPE || SLATE, "the weights' pipeline is a form of the slate step");
    constexpr uint32_t WBUF = (uint32_t)WPIPE;       // distance of the two weight buffers
    constexpr bool COPIES = LPG == 4 || LPG == 32;   // the reordered weights and sensitivities are outputs as well

    const int tid = (int)threadIdx.x;
    const int T = (int)blockDim.x;                   // a multiple of 64, at most TMAX
    const int lane = tid & 63, wave = funi(tid >> 6), nwv = T >> 6;
    const int lig = tid % LPG;
    const int mem = funi(find_matrix(wg_start, n_members, (int)blockIdx.x));
    const MatDesc &d = descs[funi(members[mem])];
    const int R = funi((int)d.rows), C = funi((int)d.cols) & ~7;   // (a multiple of the block width anyway)
    const int nbc = funi(d.nbc);
    const int opb = m >> 3;
    const int oct0 = ((int)blockIdx.x - funi(wg_start[mem])) * opu;
    const int noct = min(opu, (R >> 3) - oct0);
    const int32_t *__restrict__ rp = row_perm + d.row_off;
    const int32_t *__restrict__ cp = col_perm + d.col_off;
    const char *const Wg = reinterpret_cast<const char *>(d.w);
    const char *const Sg = reinterpret_cast<const char *>(d.s);
    const int64_t pitch_w = d.ld_w * 2, pitch_s = d.ld_s * 4;

    const uint32_t wbytes = 2u * (uint32_t)C, sbytes = 4u * (uint32_t)C;
    const int nW = (int)((wbytes + 1023u) >> 10), nS = (int)((sbytes + 1023u) >> 10);
    const uint32_t Wb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t Sb = WPIPE ? Wb + 2u * WBUF : Wb + (uint32_t)(nW * RS) * 1024u;
    float *const otab = reinterpret_cast<float *>(smem + (WPIPE ? (size_t)2 * WBUF + (size_t)nS * 1024
                                                                : (size_t)(nW + nS) * RS * 1024));   // [nbc][K] octet sums
    const int nld = nwv > 1 ? nwv - 1 : 1;           // waves that request rows
    const bool loader = wave < nld, storer = wave == nwv - 1;

    DP dp;
    dp.init(gc, lig);

    // source rows of the run (a permutation never trips the clamp; it keeps a bad one in bounds)
    for (int i = tid; i < noct * 8; i += T) {
        int sr = rp[oct0 * 8 + i];
        rowsrc[i] = sr < 0 ? 0 : (sr >= R ? R - 1 : sr);
    }

    // LDS addresses of the source columns of this lane's chunks (fixed for the whole run), row 0 of a step
    const int nchunk = C >> 3;
    uint32_t aw[CPL][8], as[SDER ? 1 : CPL][SDER ? 1 : 8];
    bool valid[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int chunk = tid + T * c;
        valid[c] = chunk < nchunk;
        const int cb = valid[c] ? chunk * 8 : 0;
        const int4 a = *reinterpret_cast<const int4 *>(cp + cb);
        const int4 b = *reinterpret_cast<const int4 *>(cp + cb + 4);
        const int t[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t sc = (uint32_t)(t[e] < 0 ? 0 : (t[e] >= C ? C - 1 : t[e]));
            aw[c][e] = Wb + (((sc >> 9) * (uint32_t)RS) << 10) + ((sc & 511u) << 1);
            if constexpr (!SDER) as[c][e] = Sb + (((sc >> 8) * (uint32_t)RS) << 10) + ((sc & 255u) << 2);
        }
    }
    const uint32_t sder = Sb - 2u * Wb;              // SDER: sensitivity address = 2 * weight address + sder
    __syncthreads();

    const int nrows = noct * 8, nrows_m1 = nrows - 1;
    // the source rows of the step that starts at `row` (read from LDS before any direct load or gather
    // read is in flight: the wait for them would otherwise wait for those as well)
    struct Rows { int sr[RS]; };
    auto source_rows = [&](int row) {
        Rows r;
#pragma unroll
        for (int rs = 0; rs < RS; ++rs) {
            int v = rowsrc[min(row + rs, nrows_m1)];
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v));           // here, not behind the gather reads issued later
            r.sr[rs] = funi(v);
        }
        return r;
    };
    auto request = [&](const Rows &r, bool do_w = true, bool do_s = true, uint32_t wbuf = 0u) {
        if (!loader) return;
#pragma unroll
        for (int rs = 0; rs < RS; ++rs)
            load_row_pieces(Wg + (int64_t)r.sr[rs] * pitch_w, Sg + (int64_t)r.sr[rs] * pitch_s, nW, nS, wbytes, sbytes,
                            Wb + wbuf, Sb, RS, rs, wave, nld, lane, do_w, do_s);
    };
    // the last wave writes the octet sums of octet `og` (in otab since the previous barrier) to part[]
    int pend_og = -1;
    auto flush = [&]() {
        if (pend_og < 0) return;
        if (storer) {
            // part: per matrix [octet of the matrix][block column][candidate], so that an octet's sums are one
            // contiguous run of whole cache lines (short writes scattered over many lines cost the read stream
            // far more than their bytes)
            float *row = part + ((d.block_base * opb + (int64_t)pend_og * nbc) * kstride + koff);
            for (int J = lane; J < nbc; J += 64) {
#pragma unroll
                for (int k = 0; k < K; ++k) row[J * kstride + k] = otab[J * K + k];
            }
        }
        pend_og = -1;
    };

    float t2[CPL][K], t3[CPL][K];                    // upper levels of the octet's row tree (B < 8 only)
    uint16_t *const wout = w_re_all + d.elem_off;
    LevelConsts lk[SUR ? CPL : 1];                   // SUR: the current grid of each chunk's block
    int curI = -1;

    // a lane's 8 reordered weights of output row orow, chunk c, as bf16 (the optional W' output)
    auto store_reordered = [&](const float (&w)[8], int orow, int c) {
        u32x4_t sv;
        sv.x = (__float_as_uint(w[0]) >> 16) | __float_as_uint(w[1]);
        sv.y = (__float_as_uint(w[2]) >> 16) | __float_as_uint(w[3]);
        sv.z = (__float_as_uint(w[4]) >> 16) | __float_as_uint(w[5]);
        sv.w = (__float_as_uint(w[6]) >> 16) | __float_as_uint(w[7]);
        __builtin_nontemporal_store(sv, (__attribute__((address_space(1))) u32x4_t *)(
                                            wout + (int64_t)orow * C + (int64_t)(tid + T * c) * 8));
    };

    // the same of the sensitivities.  (Ordinary stores: a lane has 32 bytes, so a store covers half of the lines it touches, and the
    // L2 puts the two halves together.)
    auto store_sens = [&](const float (&s)[8], int orow, int c) {
        f32x4_t *p = reinterpret_cast<f32x4_t *>(s_re_all + d.elem_off + (int64_t)orow * C + (int64_t)(tid + T * c) * 8);
        typedef __attribute__((address_space(1))) f32x4_t *gp;
        ((gp)p)[0] = f32x4_t{s[0], s[1], s[2], s[3]};
        ((gp)p)[1] = f32x4_t{s[4], s[5], s[6], s[7]};
    };

    // SLATE: one step (one row) for a wave that owns NV chunks per lane: NIT, or 1 for the last waves of a
    // workgroup whose second chunks lie past the row's end (they then skip that chunk's reads and arithmetic
    // instead of running them on nothing: with rows of 1792 chunks on 16 waves every SIMD gets 7 chunk-waves)
    constexpr bool SOLO_OK = SLATE && CPL == 2;
    const bool solo = SOLO_OK && wave * 64 + T >= nchunk;
    auto slate_step = [&](auto iu, auto inv, int row, const Rows &next, float (&t1)[CPL][K], float (&s2)[CPL][K],
                          float (&s3)[CPL][K], float (&last)[CPL][K]) {
        constexpr int u = decltype(iu)::value, NV = decltype(inv)::value;
        constexpr int NIv = DP::RP < NV ? DP::RP : NV;               // items per round of divisions
        float wv[NV][8], gs[NV][8];
        static_for<0, NV>([&](auto iit) {
            constexpr int it = decltype(iit)::value;
#pragma unroll
            for (int e = 0; e < 8; ++e) lds_w_hi<0>(wv[it][e], aw[it][e]);
        });
        static_for<0, NV>([&](auto iit) { lds_gather_wait(wv[decltype(iit)::value]); });
        asm volatile("s_barrier" ::: "memory");                      // everybody has its weights: that buffer is free
#pragma unroll
        for (int it = 0; it < NV; ++it)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t a;
                asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(a) : "v"(aw[it][e]), "s"(sder));
                gs[it][e] = *(const lds_f32 *)a;
            }
        if (row + RS < nrows) request(next, true, false);
        __builtin_amdgcn_sched_barrier(0);
        if (w_re_all) {
#pragma unroll
            for (int it = 0; it < NV; ++it)
                if (valid[it]) store_reordered(wv[it], oct0 * 8 + row, it);
        }
        // first halves of all rounds, then the sensitivities' barrier
        float xs[NV][8], vals[NV / NIv][DP::NS];
#pragma unroll
        for (int i0 = 0; i0 < NV; i0 += NIv) {
            float w[NIv][8], x[NIv][8];
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) w[j][e] = wv[i0 + j][e];
            quant_cost_prep<LPG, K, NIv, Z0>(w, dp, x, vals[i0 / NIv]);
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) xs[i0 + j][e] = x[j][e];
        }
        // (the first halves' results are operands so that their arithmetic stays above the barrier)
#pragma unroll
        for (int r = 0; r < NV / NIv; ++r)
#pragma unroll
            for (int t = 0; t < DP::NS; ++t) asm volatile("" : "+v"(vals[r][t]));
#pragma unroll
        for (int it = 0; it < NV; ++it)
            asm volatile("" : "+v"(xs[it][0]), "+v"(xs[it][1]), "+v"(xs[it][2]), "+v"(xs[it][3]),
                              "+v"(xs[it][4]), "+v"(xs[it][5]), "+v"(xs[it][6]), "+v"(xs[it][7]));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // everybody has its sensitivities
        if (row + RS < nrows) request(next, false, true);
        if constexpr (COPIES) {
#pragma unroll
            for (int it = 0; it < NV; ++it)
                if (valid[it]) store_sens(gs[it], oct0 * 8 + row, it);
        }
#pragma unroll
        for (int i0 = 0; i0 < NV; i0 += NIv) {
            float w[NIv][8], x[NIv][8], sv[NIv][8], out[NIv][K];
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) { w[j][e] = wv[i0 + j][e]; x[j][e] = xs[i0 + j][e]; sv[j][e] = gs[i0 + j][e]; }
            quant_cost_finish<LPG, K, NIv, Z0, true>(w, x, vals[i0 / NIv], sv, out);
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int k = 0; k < K; ++k) asm volatile("" : "+v"(out[j][k]));     // (see the note in the other path)
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int k = 0; k < K; ++k)
                    last[i0 + j][k] = octet_tree_push(out[j][k], u, t1[i0 + j][k], s2[i0 + j][k], s3[i0 + j][k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // WPIPE: the lane's weights of the current row (parity u of the unrolled pair) and of the next one
    float wvp[WPIPE ? 2 : 1][NIT][8];
    auto wpipe_step = [&](auto iu, auto inv, int row, const Rows &next, const Rows &next2, float (&t1)[CPL][K],
                          float (&s2)[CPL][K], float (&s3)[CPL][K], float (&last)[CPL][K]) {
        constexpr int u = decltype(iu)::value, NV = decltype(inv)::value;
        constexpr int NIv = DP::RP < NV ? DP::RP : NV;               // items per round of divisions
        constexpr int un = WPIPE ? (u ^ 1) : 0;
        float gs[NV][8];
        // the row's sensitivities out of LDS while the first half of the arithmetic runs
#pragma unroll
        for (int it = 0; it < NV; ++it)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t a;
                asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(a) : "v"(aw[it][e]), "s"(sder));
                lds_s<0>(gs[it][e], a);
            }
        if (w_re_all) {
#pragma unroll
            for (int it = 0; it < NV; ++it)
                if (valid[it]) store_reordered(wvp[u & (WPIPE ? 1 : 0)][it], oct0 * 8 + row, it);
        }
        float xs[NV][8], vals[NV / NIv][DP::NS];
#pragma unroll
        for (int i0 = 0; i0 < NV; i0 += NIv) {
            float w[NIv][8], x[NIv][8];
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) w[j][e] = wvp[u & (WPIPE ? 1 : 0)][i0 + j][e];
            quant_cost_prep<LPG, K, NIv, Z0>(w, dp, x, vals[i0 / NIv]);
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) xs[i0 + j][e] = x[j][e];
        }
#pragma unroll
        for (int r = 0; r < NV / NIv; ++r)
#pragma unroll
            for (int t = 0; t < DP::NS; ++t) asm volatile("" : "+v"(vals[r][t]));
#pragma unroll
        for (int it = 0; it < NV; ++it)
            asm volatile("" : "+v"(xs[it][0]), "+v"(xs[it][1]), "+v"(xs[it][2]), "+v"(xs[it][3]),
                              "+v"(xs[it][4]), "+v"(xs[it][5]), "+v"(xs[it][6]), "+v"(xs[it][7]));
        static_for<0, NV>([&](auto iit) { lds_gather_wait(gs[decltype(iit)::value]); });
        asm volatile("s_barrier" ::: "memory");                      // everybody has its sensitivities: that buffer is free
        if (row + 2 < nrows) request(next2, true, false, (uint32_t)u * WBUF);   // weights of row r + 2 -> the buffer row r left
        if (row + 1 < nrows) request(next, false, true);                          // sensitivities of row r + 1
        if constexpr (COPIES) {
#pragma unroll
            for (int it = 0; it < NV; ++it)
                if (valid[it]) store_sens(gs[it], oct0 * 8 + row, it);
        }
        if (row + 1 < nrows) {
            static_for<0, NV>([&](auto iit) {
                constexpr int it = decltype(iit)::value;
#pragma unroll
                for (int e = 0; e < 8; ++e) lds_w_hi<un * WBUF>(wvp[un][it][e], aw[it][e]);
            });
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i0 = 0; i0 < NV; i0 += NIv) {
            float w[NIv][8], x[NIv][8], sv[NIv][8], out[NIv][K];
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) { w[j][e] = wvp[u & (WPIPE ? 1 : 0)][i0 + j][e]; x[j][e] = xs[i0 + j][e]; sv[j][e] = gs[i0 + j][e]; }
            quant_cost_finish<LPG, K, NIv, Z0, true>(w, x, vals[i0 / NIv], sv, out);
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int k = 0; k < K; ++k) asm volatile("" : "+v"(out[j][k]));
#pragma unroll
            for (int j = 0; j < NIv; ++j)
#pragma unroll
                for (int k = 0; k < K; ++k)
                    last[i0 + j][k] = octet_tree_push(out[j][k], u, t1[i0 + j][k], s2[i0 + j][k], s3[i0 + j][k]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (row + 1 < nrows) static_for<0, NV>([&](auto iit) { lds_gather_wait(wvp[un][decltype(iit)::value]); });
    };

    request(source_rows(0));
    if constexpr (WPIPE) {
        request(source_rows(1), true, false, WBUF);                  // (nrows >= 8)
        if (loader) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        static_for<0, NIT>([&](auto iit) {
            constexpr int it = decltype(iit)::value;
#pragma unroll
            for (int e = 0; e < 8; ++e) lds_w_hi<0>(wvp[0][it][e], aw[it][e]);
        });
        static_for<0, NIT>([&](auto iit) { lds_gather_wait(wvp[0][decltype(iit)::value]); });
    }
    for (int row0 = 0; row0 < nrows; row0 += B) {
        float t1[CPL][K], s2[CPL][K], s3[CPL][K];    // static levels inside the unrolled rows
        float last[CPL][K];
        static_for<0, U>([&](auto iu) {
            constexpr int u = decltype(iu)::value;
            const int row = row0 + u * RS;           // first row of the step inside the run
            __builtin_amdgcn_sched_barrier(0);                       // (the previous step's arithmetic stays above)
            if (loader) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's share of the step's rows
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");    // everybody's: the rows are in LDS
            flush();
            const Rows next = source_rows(row + RS);                 // (clamped past the end; not requested then)
            if constexpr (SUR) {
                const int Inow = (oct0 + (row >> 3)) / opb;          // block row of this step
                if (Inow != curI) {
                    curI = Inow;
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const int J = min((tid + T * c) / LPG, nbc - 1);
                        lk[c] = level_consts(gc, level[d.block_base + (int64_t)Inow * nbc + J]);
                    }
                }
            }
            if constexpr (WPIPE) {
                const Rows next2 = source_rows(row + 2);
                if (SOLO_OK && solo) wpipe_step(iu, std::integral_constant<int, 1>{}, row, next, next2, t1, s2, s3, last);
                else wpipe_step(iu, std::integral_constant<int, NIT>{}, row, next, next2, t1, s2, s3, last);
                return;
            }
            if constexpr (SLATE) {
                if (SOLO_OK && solo) slate_step(iu, std::integral_constant<int, 1>{}, row, next, t1, s2, s3, last);
                else slate_step(iu, std::integral_constant<int, NIT>{}, row, next, t1, s2, s3, last);
                return;
            }
            // items (item = rs * CPL + c): all LDS reads of the step
            float wv[NIT][8], gs[NIT][8];
            static_for<0, NIT>([&](auto iit) {
                constexpr int it = decltype(iit)::value;
                constexpr int rs = it / CPL, c = it % CPL;
#pragma unroll
                for (int e = 0; e < 8; ++e) lds_w_hi<rs * 1024>(wv[it][e], aw[c][e]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if constexpr (SDER) {
                        uint32_t a;
                        asm volatile("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(a) : "v"(aw[c][e]), "s"(sder));
                        lds_s<rs * 1024>(gs[it][e], a);
                    } else {
                        lds_s<rs * 1024>(gs[it][e], as[c][e]);
                    }
                }
            });
            static_for<0, NIT>([&](auto iit) { lds_gather_wait(wv[decltype(iit)::value], gs[decltype(iit)::value]); });
            asm volatile("s_barrier" ::: "memory");                  // everybody has read: the buffer is free
            if (row + RS < nrows) request(next);
            __builtin_amdgcn_sched_barrier(0);

#pragma unroll
            for (int g0 = 0; g0 < NIT; g0 += NG) {
                if (w_re_all) {
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        const int rs = (g0 + g) / CPL, c = (g0 + g) % CPL;
                        if (valid[c]) store_reordered(wv[g0 + g], oct0 * 8 + row + rs, c);
                    }
                }
                if constexpr (COPIES) {
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        const int rs = (g0 + g) / CPL, c = (g0 + g) % CPL;
                        if (valid[c]) store_sens(gs[g0 + g], oct0 * 8 + row + rs, c);
                    }
                }
#pragma unroll
                for (int i0 = 0; i0 < NG; i0 += NI) {
                    float w[NI][8], s[NI][8], out[NI][K];
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int e = 0; e < 8; ++e) { w[j][e] = wv[g0 + i0 + j][e]; s[j][e] = gs[g0 + i0 + j][e]; }
                    if constexpr (SUR) {
                        LevelConsts lr[NI];
#pragma unroll
                        for (int j = 0; j < NI; ++j) lr[j] = lk[(g0 + i0 + j) % CPL];
                        surrogate_round<LPG, NI>(w, s, lr, lig, out);
                    } else {
                        quant_cost_round_f<LPG, K, NI, Z0, true>(w, s, dp, out);
                    }
                    // The sums are used by a later step's tree addition only: without an opaque use here the
                    // optimizer sinks the whole arithmetic below the next step's barriers and LDS reads
                    // (and has to keep copies of every input for it).
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(out[j][k]));
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        const int rs = (g0 + i0 + j) / CPL, c = (g0 + i0 + j) % CPL;
                        const int rr = u * RS + rs;                  // the row's place among the unrolled rows (compile time)
#pragma unroll
                        for (int k = 0; k < K; ++k) last[c][k] = octet_tree_push(out[j][k], rr, t1[c][k], s2[c][k], s3[c][k]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        });
        if constexpr (B < 8) {                       // the unrolled rows' sum enters the tree's upper levels
            static_assert(B == 2, "pairs of rows");
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (c > 0 && solo) continue;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    last[c][k] = octet_tree_push_pair_rt(last[c][k], (row0 >> 1) & 3, t2[c][k], t3[c][k]);
            }
        }

        if (((row0 + B) & 7) == 0) {                 // an octet is complete: lanes of the group, then out
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (c > 0 && solo) continue;
                float v[K];
#pragma unroll
                for (int k = 0; k < K; ++k) v[k] = group_allreduce<LPG>(last[c][k], OpAdd{});
                if (lig == 0 && valid[c]) {
                    const int J = (tid + T * c) / LPG;
#pragma unroll
                    for (int k = 0; k < K; ++k) otab[J * K + k] = v[k];
                }
            }
            pend_og = oct0 + (row0 >> 3);            // written out after the next barrier
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    flush();
}

struct FusedLaunch {
    const MatDesc *descs;
    const int *members, *wg_start;
    int n_members, total_wg;
    const int32_t *row_perm, *col_perm;
    int m;
    uint16_t *w_re;
    float *s_re;              // 32- and 256-column blocks: both copies are written; else only w_re, if not null
    float *part;
    GridConsts gc;
    int64_t cols;
    const uint8_t *level;     // surrogates only
    int kstride, koff;        // where the launch's sums go among the block's (see the kernel)
    int opu;                  // octets per workgroup of this class
};

// threads per workgroup: the chunks of a row spread over CPL per lane, rounded up to whole waves
static int fused_threads(int64_t cols, int cpl, int tmax)
{
    const int64_t need = ((cols / 8 + cpl - 1) / cpl + 63) / 64 * 64;
    return (int)(need < 64 ? 64 : (need > tmax ? tmax : need));
}

template <int LPG, int K, int CPL, int RS, int TMAX, int MINW, bool SUR, bool Z0, bool SLATE = false, int WPIPE = 0>
static int launch_fused_g(sbits_ctx *ctx, const FusedLaunch &a)
{
    int T = fused_threads(a.cols, CPL, TMAX);
    if (SLATE && T > 256) T = (T + 255) / 256 * 256 <= TMAX ? (T + 255) / 256 * 256 : T;   // whole rounds of the four SIMDs
    auto *fn = &gather_cost_kernel<LPG, K, CPL, RS, TMAX, MINW, SUR, Z0, SLATE, WPIPE>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024));
    const size_t lds = (WPIPE ? (size_t)2 * WPIPE + staged_step_bytes(a.cols, RS, true) - staged_step_bytes(a.cols, RS, false)
                              : staged_step_bytes(a.cols, RS, true)) +
                       (size_t)(a.cols / (LPG * 8)) * K * 4;                               // rows + octet sums
    hipLaunchKernelGGL(fn, dim3((unsigned)a.total_wg), dim3(T), lds, ctx->stream, a.descs, a.members,
                       a.wg_start, a.n_members, a.row_perm, a.col_perm, a.m, a.w_re, a.s_re, a.part, a.gc, a.level, a.kstride,
                       a.koff, a.opu);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

// Instances by row length (chunks of 8 columns) and candidate count:
//   up to 512 chunks : two rows per step; up to four candidates: two chunks per lane in workgroups of up
//                      to 256 threads (three workgroups = 12 waves per CU at up to 168 registers: three
//                      independent barrier groups hide each other's waits better than two of 8 waves);
//                      more candidates: one chunk per lane, up to 512 threads
//   up to 1024       : two chunks per lane, one row per step
//   up to 2048       : the same in workgroups of up to 1024 threads (one per CU: the row takes up to
//                      96 KB of LDS)
template <int LPG, int K, bool Z0>
static int launch_fused_k(sbits_ctx *ctx, const FusedLaunch &a)
{
    const int64_t chunks = a.cols / 8;
    constexpr int MINW = K <= 4 ? 4 : 2;             // waves per SIMD the register budget is set for
    if (chunks <= 512) {
        // (two chunks and two rows per lane where that fits 168 registers without spilling; else one chunk of one
        // row, 62 to 82 registers: three workgroups per CU; measured 2 to 6 % faster than two rows per step there)
        if constexpr (K <= 2 || (K <= 4 && !Z0 && LPG >= 16)) return launch_fused_g<LPG, K, 2, 2, 256, 3, false, Z0>(ctx, a);
        // (... as long as it stays within the 80 registers that three workgroups of eight waves leave a lane)
        else if constexpr (LPG >= 16 ? (K <= 7 || (K == 8 && !Z0)) : (K <= 5 || (K == 6 && !Z0)))
            return launch_fused_g<LPG, K, 1, 1, 512, 4, false, Z0>(ctx, a);
        else return launch_fused_g<LPG, K, 1, 2, 512, MINW, false, Z0>(ctx, a);
    }
    if (chunks <= 1024) return launch_fused_g<LPG, K, 2, 1, 512, MINW, false, Z0>(ctx, a);
    if (chunks <= 2048) {
        // seven or more candidates: two chunks' state does not fit the 128 registers of a 1024-thread workgroup
        // the slate form; with the weights pipelined where that fits the 128 registers (or nearly: 16 bytes of
        // scratch at five candidates still pay, 24 and more do not)
        if constexpr (LPG == 16 ? K <= 5 : LPG > 16 ? K <= 4 : (K <= 2 || (K == 3 && !Z0)))
            return launch_fused_g<LPG, K, 2, 1, 1024, 4, false, Z0, true, 32768>(ctx, a);
        else if constexpr (K <= 5 || (K == 6 && !(Z0 && LPG <= 8))) return launch_fused_g<LPG, K, 2, 1, 1024, 4, false, Z0, true>(ctx, a);
        else return launch_fused_g<LPG, K, 2, 1, 1024, 4, false, Z0, false>(ctx, a);
    }
    return SBITS_ERR_BAD_SHAPE;
}

// K: the candidates of this launch; z0: the first of them is 0 bits (then 2 <= K <= 9, else 1 <= K <= 8)
template <int LPG>
static int launch_fused_l(int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a)
{
    if (z0) switch (K) {
    case 2: return launch_fused_k<LPG, 2, true>(ctx, a);
    case 3: return launch_fused_k<LPG, 3, true>(ctx, a);
    case 4: return launch_fused_k<LPG, 4, true>(ctx, a);
    case 5: return launch_fused_k<LPG, 5, true>(ctx, a);
    case 6: return launch_fused_k<LPG, 6, true>(ctx, a);
    case 7: return launch_fused_k<LPG, 7, true>(ctx, a);
    case 8: return launch_fused_k<LPG, 8, true>(ctx, a);
    case 9: return launch_fused_k<LPG, 9, true>(ctx, a);
    }
    else switch (K) {
    case 1: return launch_fused_k<LPG, 1, false>(ctx, a);
    case 2: return launch_fused_k<LPG, 2, false>(ctx, a);
    case 3: return launch_fused_k<LPG, 3, false>(ctx, a);
    case 4: return launch_fused_k<LPG, 4, false>(ctx, a);
    case 5: return launch_fused_k<LPG, 5, false>(ctx, a);
    case 6: return launch_fused_k<LPG, 6, false>(ctx, a);
    case 7: return launch_fused_k<LPG, 7, false>(ctx, a);
    case 8: return launch_fused_k<LPG, 8, false>(ctx, a);
    }
    return SBITS_ERR_BAD_BITWIDTHS;
}

}  // namespace sbits
