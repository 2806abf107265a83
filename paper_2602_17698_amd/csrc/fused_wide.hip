// Reorder-gather fused with the cost table for rows of more than 16384 elements, whose weights and sensitivities (6 bytes an element, up to
// 192 KiB) do not fit LDS together.  The same operation, arithmetic and order of sums as gather_cost_kernel.
//
// PARTS workgroups share a row: each stages all of it and scores its part of the output columns, CPL chunks of 8 per lane.  They are eight apart in
// the grid, so that they share an L2 and walk the same rows at the same time.  A row passes through LDS in two overlapping
// halves of a step:
//   pieces (1 KiB)   sensitivities 0 .. nS, weights w0 .. w0 + nW with w0 = nS - O: the last O pieces of the sensitivities and the first O of
//                    the weights have the same place, O as small as the room beside the octet sums allows (none up to 26880 elements at
//                    one candidate, up to 25600 at nine in 64-column blocks and two parts; a dozen for 28672, 34 to 42 for 32768)
//   weights out of LDS | barrier | request the O late pieces of the sensitivities | minimum, range, divisions, x = w - min
//   | wait, barrier | request the next row's weights but the first O | sensitivities out of LDS | barrier | request the next
//   row's sensitivities but the last O, and its first O weights | candidates, sums | wait, barrier
// What bounds it is a step's chain of four barriers with one workgroup a CU, between which only the last stretch has much arithmetic: 5.8 us a
// row of 28672 and two parts at three candidates.  The loads are ordinary ones (the other parts want the row from the L2; nontemporal: the
// same within 3 % either way).  8192 x 28672, three candidates: 374 us, where reordering the row into memory, 18 bytes an element in all, and scoring that
// took 740; five candidates in 64-column blocks 846 -> 411, eight 926 -> 495, 20480 x 17408 1116 -> 654.
#include "fused_core.hpp"

namespace sbits {

constexpr int FW_THREADS = 1024;
constexpr int FW_LDS = 159 * 1024;                  // rows and octet sums

template <int LPG, int K, int CPL, bool Z0>
__global__ __launch_bounds__(FW_THREADS, 4)
void gather_cost_wide_kernel(const MatDesc *__restrict__ descs, const int *__restrict__ members, const int *__restrict__ wg_start, int n_members,
                             const int32_t *__restrict__ row_perm, const int32_t *__restrict__ col_perm, int m, uint16_t *__restrict__ w_re_all,
                             float *__restrict__ part, GridConsts gc, int opu, int overlap)
{
    constexpr int PARTS = 4 / CPL;
    static_assert(CPL == 1 || CPL == 2, "four chunks a lane between the parts");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int rowsrc[FU_OPU * 8];
    using DP = DivPlan<LPG, K - Z0>;
    constexpr int NI = DP::RP < CPL ? DP::RP : CPL;  // chunks that share a round of divisions

    const int tid = (int)threadIdx.x, T = (int)blockDim.x;
    const int lane = tid & 63, wave = funi(tid >> 6), nwv = T >> 6;
    const int lig = tid % LPG;
    const int unit = (int)(blockIdx.x / (8 * PARTS) * 8 + (blockIdx.x & 7)), my_part = (int)(blockIdx.x >> 3) % PARTS;
    if (unit >= funi(wg_start[n_members])) return;
    const int mem = funi(find_matrix(wg_start, n_members, unit));
    const MatDesc &d = descs[funi(members[mem])];
    const int R = funi((int)d.rows), C = funi((int)d.cols) & ~7;
    const int nbc = funi(d.nbc);
    const int opb = m >> 3;
    const int oct0 = (unit - funi(wg_start[mem])) * opu;
    const int noct = min(opu, (R >> 3) - oct0);
    const int32_t *__restrict__ rp = row_perm + d.row_off;
    const int32_t *__restrict__ cp = col_perm + d.col_off;
    const char *const Wg = reinterpret_cast<const char *>(d.w);
    const char *const Sg = reinterpret_cast<const char *>(d.s);
    const int64_t pitch_w = d.ld_w * 2, pitch_s = d.ld_s * 4;

    const uint32_t wbytes = 2u * (uint32_t)C, sbytes = 4u * (uint32_t)C;
    const int nW = (int)((wbytes + 1023u) >> 10), nS = (int)((sbytes + 1023u) >> 10);
    const uint32_t Sb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t Wb = Sb + (uint32_t)(nS - overlap) * 1024u;
    const int chunk0 = my_part * CPL * T, nchunk = C >> 3;
    const int J0 = chunk0 / LPG, nJ = min(nbc - J0, CPL * T / LPG);          // this part's block columns (0 or less: none)
    float *const otab = reinterpret_cast<float *>(smem + (size_t)(nS + nW - overlap) * 1024);    // [block column][K] octet sums
    const int nld = nwv - 1;                         // waves that request rows; the last one stores
    const bool loader = wave < nld, storer = wave == nld;

    DP dp;
    dp.init(gc, lig);
    for (int i = tid; i < noct * 8; i += T) {
        int sr = rp[oct0 * 8 + i];
        rowsrc[i] = sr < 0 ? 0 : (sr >= R ? R - 1 : sr);
    }
    uint32_t aw[CPL][8];                             // LDS addresses of the weights of this lane's source columns
    bool valid[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int chunk = chunk0 + tid + T * c;
        valid[c] = chunk < nchunk;
        const int cb = valid[c] ? chunk * 8 : 0;
        const int4 a = *reinterpret_cast<const int4 *>(cp + cb);
        const int4 b = *reinterpret_cast<const int4 *>(cp + cb + 4);
        const int t[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t sc = (uint32_t)(t[e] < 0 ? 0 : (t[e] >= C ? C - 1 : t[e]));
            aw[c][e] = Wb + (sc << 1);
        }
    }
    const uint32_t sder = Sb - 2u * Wb;              // sensitivity address = 2 * weight address + sder
    __syncthreads();

    const int nrows = noct * 8;
    auto source_row = [&](int row) {
        int v = rowsrc[min(row, nrows - 1)];
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v));
        return funi(v);
    };
    // pieces p0 .. p1 of a row, between the loading waves
    auto request = [&](const char *row, uint32_t bytes, uint32_t base, int p0, int p1) {
        if (!loader) return;
        for (int p = p0 + wave; p < p1; p += nld) {
            const uint32_t off = min((uint32_t)p * 1024u + (uint32_t)lane * 16u, bytes - 16u);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + off),
                                             (__attribute__((address_space(3))) void *)(base + (uint32_t)p * 1024u), 16, 0, 0);
        }
    };
    auto rows_there = [&]() {
        if (loader) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    int pend_og = -1;                                // the octet whose sums are in otab since the previous barrier
    auto flush = [&]() {
        if (pend_og < 0) return;
        if (storer) {
            float *row = part + ((d.block_base * opb + (int64_t)pend_og * nbc + J0) * K);
            for (int i = lane; i < nJ * K; i += 64) row[i] = otab[i];
        }
        pend_og = -1;
    };
    uint16_t *const wout = w_re_all + d.elem_off;
    float t2[CPL][K], t3[CPL][K];                    // upper levels of the octet's row tree

    {
        const int64_t sr = source_row(0);
        request(Wg + sr * pitch_w, wbytes, Wb, 0, nW);
        request(Sg + sr * pitch_s, sbytes, Sb, 0, nS - overlap);
    }
    for (int row0 = 0; row0 < nrows; row0 += 2) {
        float t1[CPL][K], s2[CPL][K], s3[CPL][K], last[CPL][K];
        static_for<0, 2>([&](auto iu) {
            constexpr int u = decltype(iu)::value;
            const int row = row0 + u;
            __builtin_amdgcn_sched_barrier(0);
            rows_there();
            flush();
            const int64_t sr = source_row(row), next = source_row(row + 1);
            float w[CPL][8];
            static_for<0, CPL>([&](auto ic) {
                constexpr int c = decltype(ic)::value;
#pragma unroll
                for (int e = 0; e < 8; ++e) lds_w_hi<0>(w[c][e], aw[c][e]);
            });
            static_for<0, CPL>([&](auto ic) { lds_gather_wait(w[decltype(ic)::value]); });
            asm volatile("s_barrier" ::: "memory");                      // everybody has its weights: their place is free
            request(Sg + sr * pitch_s, sbytes, Sb, nS - overlap, nS);
            __builtin_amdgcn_sched_barrier(0);
            if (w_re_all) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    if (!valid[c]) continue;
                    u32x4_t sv;
                    sv.x = (__float_as_uint(w[c][0]) >> 16) | __float_as_uint(w[c][1]);
                    sv.y = (__float_as_uint(w[c][2]) >> 16) | __float_as_uint(w[c][3]);
                    sv.z = (__float_as_uint(w[c][4]) >> 16) | __float_as_uint(w[c][5]);
                    sv.w = (__float_as_uint(w[c][6]) >> 16) | __float_as_uint(w[c][7]);
                    __builtin_nontemporal_store(sv, (__attribute__((address_space(1))) u32x4_t *)(
                                                        wout + (int64_t)(oct0 * 8 + row) * C + (int64_t)(chunk0 + tid + T * c) * 8));
                }
            }
            float xs[CPL][8], vals[CPL / NI][DP::NS];
#pragma unroll
            for (int i0 = 0; i0 < CPL; i0 += NI) {
                float wi[NI][8], x[NI][8];
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) wi[j][e] = w[i0 + j][e];
                quant_cost_prep<LPG, K, NI, Z0>(wi, dp, x, vals[i0 / NI]);
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) xs[i0 + j][e] = x[j][e];
            }
            // (operands here, so that the arithmetic stays above the barrier)
#pragma unroll
            for (int r = 0; r < CPL / NI; ++r)
#pragma unroll
                for (int t = 0; t < DP::NS; ++t) asm volatile("" : "+v"(vals[r][t]));
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                asm volatile("" : "+v"(xs[c][0]), "+v"(xs[c][1]), "+v"(xs[c][2]), "+v"(xs[c][3]),
                                  "+v"(xs[c][4]), "+v"(xs[c][5]), "+v"(xs[c][6]), "+v"(xs[c][7]));
            rows_there();                                                // the row's sensitivities are whole
            if (row + 1 < nrows) request(Wg + next * pitch_w, wbytes, Wb, overlap, nW);
            float gs[CPL][8];
            static_for<0, CPL>([&](auto ic) {
                constexpr int c = decltype(ic)::value;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    uint32_t a;
                    asm volatile("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(a) : "v"(aw[c][e]), "s"(sder));
                    lds_s<0>(gs[c][e], a);
                }
            });
            static_for<0, CPL>([&](auto ic) { lds_gather_wait(gs[decltype(ic)::value]); });
            asm volatile("s_barrier" ::: "memory");                      // everybody has its sensitivities
            if (row + 1 < nrows) {
                request(Sg + next * pitch_s, sbytes, Sb, 0, nS - overlap);
                request(Wg + next * pitch_w, wbytes, Wb, 0, overlap);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i0 = 0; i0 < CPL; i0 += NI) {
                float wi[NI][8], x[NI][8], sv[NI][8], out[NI][K];
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) { wi[j][e] = w[i0 + j][e]; x[j][e] = xs[i0 + j][e]; sv[j][e] = gs[i0 + j][e]; }
                quant_cost_finish<LPG, K, NI, Z0, true>(wi, x, vals[i0 / NI], sv, out);
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(out[j][k]));
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        last[i0 + j][k] = octet_tree_push(out[j][k], u, t1[i0 + j][k], s2[i0 + j][k], s3[i0 + j][k]);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) last[c][k] = octet_tree_push_pair_rt(last[c][k], (row0 >> 1) & 3, t2[c][k], t3[c][k]);
        if (((row0 + 2) & 7) == 0) {                 // an octet is complete: lanes of the group, then out
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
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

template <int LPG, int K, int CPL, bool Z0>
static int launch_wide_g(sbits_ctx *ctx, const FusedLaunch &a)
{
    constexpr int PARTS = 4 / CPL;
    int T = fused_threads(a.cols, CPL * PARTS, FW_THREADS);
    T = (T + 255) / 256 * 256;                       // whole rounds of the four SIMDs
    const int nW = (int)((2 * a.cols + 1023) / 1024), nS = (int)((4 * a.cols + 1023) / 1024);
    const int sums = (CPL * T / LPG) * K * 4, room = (FW_LDS - sums) / 1024;
    const int overlap = nW + nS > room ? nW + nS - room : 0;
    auto *fn = &gather_cost_wide_kernel<LPG, K, CPL, Z0>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, FW_LDS));
    const size_t lds = (size_t)(nW + nS - overlap) * 1024 + (size_t)sums;
    hipLaunchKernelGGL(fn, dim3(((unsigned)a.total_wg + 7u) / 8u * 8u * PARTS), dim3(T), lds, ctx->stream, a.descs, a.members, a.wg_start, a.n_members,
                       a.row_perm, a.col_perm, a.m, a.w_re, a.part, a.gc, a.opu, overlap);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

// Four parts, with half of the work a step, while all workgroups are on the chip at once even so: 256 x 28672 at three candidates 48 us
// with two, 35 with four (in two passes, as before, 39); 768 x 28672 48 and 58.  (Two chunks a lane spill up to 92 bytes at eight and
// nine candidates and are the faster form all the same: 8192 x 32768 in 64-column blocks at nine 709 us with one, 593 with two.)
template <int LPG, int K, bool Z0>
static int launch_wide_k(sbits_ctx *ctx, const FusedLaunch &a)
{
    return a.total_wg * 4 <= sbits_cus(ctx) ? launch_wide_g<LPG, K, 1, Z0>(ctx, a) : launch_wide_g<LPG, K, 2, Z0>(ctx, a);
}

template <int LPG>
static int launch_wide_l(int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a)
{
    if (z0) switch (K) {
    case 2: return launch_wide_k<LPG, 2, true>(ctx, a);
    case 3: return launch_wide_k<LPG, 3, true>(ctx, a);
    case 4: return launch_wide_k<LPG, 4, true>(ctx, a);
    case 5: return launch_wide_k<LPG, 5, true>(ctx, a);
    case 6: return launch_wide_k<LPG, 6, true>(ctx, a);
    case 7: return launch_wide_k<LPG, 7, true>(ctx, a);
    case 8: return launch_wide_k<LPG, 8, true>(ctx, a);
    case 9: return launch_wide_k<LPG, 9, true>(ctx, a);
    }
    else switch (K) {
    case 1: return launch_wide_k<LPG, 1, false>(ctx, a);
    case 2: return launch_wide_k<LPG, 2, false>(ctx, a);
    case 3: return launch_wide_k<LPG, 3, false>(ctx, a);
    case 4: return launch_wide_k<LPG, 4, false>(ctx, a);
    case 5: return launch_wide_k<LPG, 5, false>(ctx, a);
    case 6: return launch_wide_k<LPG, 6, false>(ctx, a);
    case 7: return launch_wide_k<LPG, 7, false>(ctx, a);
    case 8: return launch_wide_k<LPG, 8, false>(ctx, a);
    }
    return SBITS_ERR_BAD_BITWIDTHS;
}

}  // namespace sbits

using namespace sbits;

int sbits_launch_fused_wide(int n, int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a)
{
    return n == 64 ? launch_wide_l<8>(K, z0, ctx, a) : launch_wide_l<16>(K, z0, ctx, a);
}
