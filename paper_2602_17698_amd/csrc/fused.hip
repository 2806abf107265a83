// Reorder-gather fused with the block x bitwidth cost table: the original weights (bf16) and
// sensitivities (fp32) are read ONCE, permuted on the fly and scored; the reordered weights are
// written back only if the caller asks for them (the packing stage reads the originals too).  The
// reordered sensitivities never reach HBM.
//
// Operation: the same as gather followed by the cost table (paper Sec. 4.2 "bi-directional
// channel reordering" applied to W and S, then Sec. 5 "Implementation": per-block-row
// round-to-nearest grids for every candidate bitwidth), with the same fixed summation order,
// so the table equals the two-pass result bit for bit.
//
// Mapping.  A workgroup owns a run of octets (8 output rows each) of one matrix, all columns.
// Per step it has RS source rows (the rows row_perm names) brought into LDS by direct
// global-to-LDS loads (no registers in between), then every lane picks the 8 source columns of
// each of its CPL output chunks (chunk = 8 consecutive output columns; LPG adjacent lanes = one
// quantization group) out of LDS and scores them while the next step's rows are on their way.
// The levels of the octet's row tree are compile-time positions of an unrolled run of steps; at
// the end of an octet the group's lanes are reduced and the octet's partial sum goes to
// part[octet of the matrix][block column][candidate]; a second, tiny kernel runs the tree over the
// octets of each block.
#include "fused_core.hpp"

namespace sbits {

// adjacent-pair tree over n <= 8 values p[0], p[stride], ... (n a power of two)
__device__ __forceinline__ float tree_upto8(const float *__restrict__ p, int64_t stride, int n)
{
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = i < n ? p[i * stride] : 0.0f;
    if (n == 1) return v[0];
    if (n == 2) return v[0] + v[1];
    if (n == 4) return (v[0] + v[1]) + (v[2] + v[3]);
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// Where the octet sums of global block b start in part[] (layout per matrix: [octet][block column][sum], ks sums
// per entry) and the distance between consecutive octets of the block.  The matrix is found by bisection over the
// descriptors' first block ids.
__device__ __forceinline__ const float *block_partials(const float *__restrict__ part, const MatDesc *__restrict__ descs,
                                                       int n_mats, int64_t b, int opb, int ks, int64_t *stride)
{
    int lo = 0, hi = n_mats;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (descs[mid].block_base <= b) lo = mid; else hi = mid;
    }
    const int64_t base = descs[lo].block_base;
    const int nbc = descs[lo].nbc;
    const int64_t bl = b - base;
    const int64_t I = bl / nbc, J = bl - I * nbc;
    *stride = (int64_t)nbc * ks;
    return part + (base * opb + I * opb * nbc + J) * ks;
}

// cost[b][c] = adjacent-pair tree over the opb octet partials of block b (opb a power of two <= 128)
__global__ __launch_bounds__(256)
void octet_finish_kernel(const float *__restrict__ part, const MatDesc *__restrict__ descs, int n_mats, int64_t NK,
                         int K, int opb, float *__restrict__ cost)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= NK) return;
    const int64_t b = q / K;
    const int c = (int)(q - b * K);
    int64_t so;                                      // distance between the block's consecutive octets
    const float *p = block_partials(part, descs, n_mats, b, opb, K, &so) + c;
    if (opb <= 8) {
        cost[q] = tree_upto8(p, so, opb);
        return;
    }
    float t1 = 0.0f, t2 = 0.0f, t3 = 0.0f, t4 = 0.0f, v = 0.0f;
    const int ng = opb >> 3;                         // 2 .. 16 groups of 8 octets
    for (int g = 0; g < ng; ++g) {
        v = tree_upto8(p + (int64_t)g * 8 * so, so, 8);
        if (g & 1) {
            v = t1 + v;
            if (g & 2) {
                v = t2 + v;
                if (g & 4) {
                    v = t3 + v;
                    if (g & 8) v = t4 + v;
                    else t4 = v;
                } else {
                    t3 = v;
                }
            } else {
                t2 = v;
            }
        } else {
            t1 = v;
        }
    }
    cost[q] = v;
}

// ================================================================ gather + pack
// The packing stage on the ORIGINAL weights: a workgroup owns a run of octets of one matrix,
// stages RS source rows per step in LDS like the kernel above (weights only), and every lane
// re-quantizes its chunks at the bitwidth chosen for their block.  The codes of four rows of a lane
// group, from one step or from two, are consecutive in the block's stream and leave as whole words
// (store_codes4).  WIDE: a candidate has more than 4 bits.
// Rows go through registers into one of two LDS buffers, in the cost kernel's layout, and a lane takes its elements out as floats (upper
// halves): one barrier a step, no packing and unpacking.  (Awaiting the next rows before a step's stores, or less rows a step for
// more waves: 3 to 7 % slower.)
// T threads per workgroup; launch bounds ask for 4 waves per SIMD (two workgroups of 512 or one
// of 1024 per CU), which the kernel's ~120 registers allow.
// PARTS = 2 (rows of more than 16384 elements): two workgroups stage the same rows and pack half of the columns each, two chunks
// per lane as for shorter rows; they are eight apart in the grid, so that they share an L2.  (All columns in one workgroup are
// four chunks a lane, one row a step, 33 registers spilled: 8192 x 28672 in 382 us, 202 this way.)
// MASK: for a device whose 16-bit loads leave the other half of the register as it was (see lds_w_hi); not for the others, because it
// costs an AND per weight.
template <int LPG, int CPL, int RS, int TMAX, bool WIDE, int PARTS = 1, bool MASK = false>
__global__ __launch_bounds__(TMAX, 4)
void gather_pack_kernel(const MatDesc *__restrict__ descs, const int *__restrict__ members,
                        const int *__restrict__ wg_start, int n_members,
                        const int32_t *__restrict__ row_perm, const int32_t *__restrict__ col_perm, int m,
                        const uint8_t *__restrict__ level, const int64_t *__restrict__ byte_off,
                        uint8_t *__restrict__ codes, float *__restrict__ scale, float *__restrict__ zero,
                        GridConsts gc, int opu, const unsigned *__restrict__ aborted)
{
    const unsigned stop = aborted ? *aborted : 0u;   // the levels are those of a search that gave up: not used
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int rowsrc[FU_OPU * 8];
    constexpr int NIT = RS * CPL;
    static_assert(RS == 2 || RS == 4, "a group of four rows is one step or two");

    const int tid = (int)threadIdx.x;
    const int T = (int)blockDim.x;                   // a multiple of 64, at most TMAX
    const int lig = tid % LPG;
    const int unit = PARTS == 1 ? (int)blockIdx.x : (int)(blockIdx.x >> 4 << 3 | (blockIdx.x & 7));
    if (PARTS > 1 && unit >= wg_start[n_members]) return;
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
    const int64_t pitch_w = d.ld_w * 2;
    const int64_t block_base = d.block_base;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;    // weights [RS][C] bf16
    for (int i = tid; i < noct * 8; i += T) {
        int sr = rp[oct0 * 8 + i];
        rowsrc[i] = sr < 0 ? 0 : (sr >= R ? R - 1 : sr);
    }
    const int nchunk = C >> 3;
    const int chunk0 = PARTS == 1 ? 0 : (int)(blockIdx.x >> 3 & 1) * CPL * T;    // this workgroup's chunks: CPL * T from here (whole groups)
    uint32_t ci[CPL][8];                             // LDS addresses of the source columns, row 0 of a step in the first buffer
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
            ci[c][e] = lds0 + (((sc >> 9) * (uint32_t)RS) << 10) + ((sc & 511u) << 1);
        }
    }
    __syncthreads();

    constexpr int STG = CPL * PARTS;                 // chunks that a lane stages of a row
    uint32_t offw[STG];
#pragma unroll
    for (int c = 0; c < STG; ++c) offw[c] = (uint32_t)min(tid + T * c, nchunk - 1) * 16u;
    uint4 pw[RS][STG];
    auto prefetch = [&](int row) {
#pragma unroll
        for (int rs = 0; rs < RS; ++rs) {
            const int sr = funi(rowsrc[row + rs]);
            const char *wrow = Wg + (int64_t)sr * pitch_w;
#pragma unroll
            for (int c = 0; c < STG; ++c) {
                const __attribute__((address_space(1))) u32x4_t *p = (const __attribute__((address_space(1))) u32x4_t *)(wrow + offw[c]);
                const u32x4_t v = PARTS == 1 ? __builtin_nontemporal_load(p) : *p;           // (the other workgroup reads it too)
                pw[rs][c] = make_uint4(v.x, v.y, v.z, v.w);
            }
        }
    };
    // Rows lie piece by piece (1 KiB), the rows of a step interleaved, as in the cost kernel; two buffers where they fit.
    constexpr bool TWO = PARTS == 1;
    const uint32_t buffer = (uint32_t)((2 * C + 1023) >> 10) * (uint32_t)RS << 10;
    auto stage = [&](uint32_t buf) {
#pragma unroll
        for (int rs = 0; rs < RS; ++rs)
#pragma unroll
            for (int c = 0; c < STG; ++c)
                *reinterpret_cast<uint4 *>(smem + buf + (((offw[c] >> 10) * RS + rs) << 10) + (offw[c] & 1023u)) = pw[rs][c];
    };

    // per chunk: the block it falls in (fixed column, block row changes every opb octets)
    int curI = -1;
    LevelConsts lk[CPL];
    int64_t gb[CPL];
    uint8_t *dst[CPL];
    const int nsteps = noct * (8 / RS);

    uint32_t held_lo[RS == 4 ? 1 : CPL][4], held_hi[RS == 4 ? 1 : CPL][4];     // rows that wait for the rest of their four
    prefetch(0);
    if (stop) return;
    if constexpr (TWO) {
        stage(0u);
        if (nsteps > 1) prefetch(RS);
    }
    uint32_t buf = 0u;
    for (int st = 0; st < nsteps; ++st) {
        if constexpr (TWO) {
            lds_barrier();                           // this step's rows are there, the other buffer has been read
            if (st + 1 < nsteps) stage(buffer - buf);
            if (st + 2 < nsteps) prefetch((st + 2) * RS);
        } else {
            stage(0u);
            lds_barrier();
            if (st + 1 < nsteps) prefetch((st + 1) * RS);
        }

        const int row = st * RS;
        const int og = oct0 + (row >> 3);
        const int I = og / opb;
        const int rib = (og - I * opb) * 8 + (row & 7);         // first row of the step inside its block
        if (I != curI) {
            curI = I;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int J = min((chunk0 + tid + T * c) / LPG, nbc - 1);
                gb[c] = block_base + (int64_t)I * nbc + J;
                lk[c] = level_consts(gc, level[gb[c]]);
                dst[c] = codes + byte_off[gb[c]];
            }
        }

        float gw[TWO ? RS : NIT][8];
        auto gather = [&](auto ic) {                 // the lane's elements of chunk c, rows of the step
            constexpr int c = decltype(ic)::value, at = TWO ? 0 : c * RS;
            static_for<0, RS>([&](auto irs) {
                constexpr int rs = decltype(irs)::value;
#pragma unroll
                for (int e = 0; e < 8; ++e) lds_w_hi<rs * 1024>(gw[at + rs][e], ci[c][e] + buf);
            });
        };
        if constexpr (!TWO) {
            static_for<0, CPL>([&](auto ic) { gather(ic); });
            static_for<0, NIT>([&](auto iit) { lds_gather_wait(gw[decltype(iit)::value]); });
            asm volatile("s_barrier" ::: "memory");  // the rows may be overwritten from here on
        }

        static_for<0, CPL>([&](auto ic) {
            constexpr int c = decltype(ic)::value;
            if constexpr (TWO) {
                gather(ic);
                static_for<0, RS>([&](auto irs) { lds_gather_wait(gw[decltype(irs)::value]); });
            }
            const int cb = lk[c].c;
            float w[RS][8];
#pragma unroll
            for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    w[rs][e] = gw[(TWO ? 0 : c * RS) + rs][e];
                    if constexpr (MASK) w[rs][e] = __uint_as_float(__float_as_uint(w[rs][e]) & 0xffff0000u);
                }
            uint32_t half[RS][2];
            float scl[RS], mn[RS];
            quant_pack_rows<LPG, RS>(w, lk[c], lig, half, scl, mn);
            uint32_t lo[RS], hi[RS];
#pragma unroll
            for (int rs = 0; rs < RS; ++rs) {
                if constexpr (WIDE) {
                    const uint64_t w = (uint64_t)half[rs][1] << (4 * cb) | half[rs][0];
                    lo[rs] = (uint32_t)w;
                    hi[rs] = (uint32_t)(w >> 32);
                } else {
                    lo[rs] = half[rs][1] << (4 * cb) | half[rs][0];
                    hi[rs] = 0u;
                }
            }
            if (valid[c] && lig == 0) {
                // RS consecutive rows of one block: one vector store each (rib is a multiple of RS)
                const int64_t ri = gb[c] * m + rib;
                float zr[RS];
#pragma unroll
                for (int rs = 0; rs < RS; ++rs) zr[rs] = mn[rs] + 0.0f;
                if constexpr (RS == 4) {
                    *reinterpret_cast<float4 *>(scale + ri) = make_float4(scl[0], scl[1], scl[2], scl[3]);
                    *reinterpret_cast<float4 *>(zero + ri) = make_float4(zr[0], zr[1], zr[2], zr[3]);
                } else {
                    *reinterpret_cast<float2 *>(scale + ri) = make_float2(scl[0], scl[1]);
                    *reinterpret_cast<float2 *>(zero + ri) = make_float2(zr[0], zr[1]);
                }
            }
            // the rows of this step, behind those of the steps before it in the same group of four
            uint8_t *const out = dst[c] + (int64_t)(rib & ~3) * (LPG * cb);
            if constexpr (RS == 4) {
                if (valid[c]) store_codes4<LPG, WIDE>(out, cb, lo, hi, lig);
            } else {
#pragma unroll
                for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (q % RS == rs && (rib & 3) == q - rs) { held_lo[c][q] = lo[rs]; held_hi[c][q] = hi[rs]; }
                if ((rib & 3) == 4 - RS && valid[c]) store_codes4<LPG, WIDE>(out, cb, held_lo[c], held_hi[c], lig);
            }
        });
        if constexpr (TWO) buf = buffer - buf;
    }
}

// surrogates: s_up[b] = tree over the octets of sum 0, s_down[b] = 2^-bits * tree over those of sum 1
__global__ __launch_bounds__(256)
void surrogate_finish_kernel(const float *__restrict__ part, const MatDesc *__restrict__ descs, int n_mats, int64_t N,
                             int opb, const uint8_t *__restrict__ level, GridConsts gc, float *__restrict__ s_up,
                             float *__restrict__ s_down)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= 2 * N) return;
    const int64_t b = q >> 1;
    const int which = (int)(q & 1);
    int64_t so;
    const float *p = block_partials(part, descs, n_mats, b, opb, 2, &so) + which;
    float v;
    if (opb <= 8) {
        v = tree_upto8(p, so, opb);
    } else {
        float t1 = 0.0f, t2 = 0.0f, t3 = 0.0f, t4 = 0.0f;
        v = 0.0f;
        const int ng = opb >> 3;
        for (int g = 0; g < ng; ++g) {
            v = tree_upto8(p + (int64_t)g * 8 * so, so, 8);
            if (g & 1) {
                v = t1 + v;
                if (g & 2) {
                    v = t2 + v;
                    if (g & 4) {
                        v = t3 + v;
                        if (g & 8) v = t4 + v;
                        else t4 = v;
                    } else {
                        t3 = v;
                    }
                } else {
                    t2 = v;
                }
            } else {
                t1 = v;
            }
        }
    }
    if (which == 0) {
        s_up[b] = v;
    } else {
        int bits = gc.bits[0];
#pragma unroll
        for (int cc = 1; cc < MAX_CAND; ++cc)
            if (level[b] == cc) bits = gc.bits[cc];
        s_down[b] = ldexpf(v, -bits);
    }
}

template <int LPG>
static int launch_surrogates_l(sbits_ctx *ctx, const FusedLaunch &a)
{
    const int64_t chunks = a.cols / 8;
    if (chunks <= 512) return launch_fused_g<LPG, 2, 1, 2, 512, 4, true, false>(ctx, a);
    if (chunks <= 1024) return launch_fused_g<LPG, 2, 2, 1, 512, 4, true, false>(ctx, a);
    if (chunks <= 2048) return launch_fused_g<LPG, 2, 2, 1, 1024, 4, true, false>(ctx, a);
    return SBITS_ERR_BAD_SHAPE;
}

struct FusedPackLaunch {
    const MatDesc *descs;
    const int *members, *wg_start;
    int n_members, total_wg;
    const int32_t *row_perm, *col_perm;
    int m;
    const uint8_t *level;
    const int64_t *byte_off;
    uint8_t *codes;
    float *scale, *zero;
    GridConsts gc;
    bool wide;                // a candidate has more than 4 bits
    bool mask;                // 16-bit loads into a register half leave the other one as it was
    int64_t cols;
    int opu;
    const unsigned *aborted;
};

template <int LPG, int CPL, int RS, int TMAX, int PARTS = 1>
static int launch_gpack_g(sbits_ctx *ctx, const FusedPackLaunch &a)
{
    const int T = fused_threads(a.cols, CPL * PARTS, TMAX);
    auto *fn = a.mask ? &gather_pack_kernel<LPG, CPL, RS, TMAX, true, PARTS, true>
             : a.wide ? &gather_pack_kernel<LPG, CPL, RS, TMAX, true, PARTS> : &gather_pack_kernel<LPG, CPL, RS, TMAX, false, PARTS>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024));
    const size_t lds = (PARTS == 1 ? 2 : 1) * staged_step_bytes(a.cols, RS, false);
    const unsigned grid = PARTS == 1 ? (unsigned)a.total_wg : ((unsigned)a.total_wg + 7u) / 8u * 16u;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(T), lds, ctx->stream, a.descs, a.members,
                       a.wg_start, a.n_members, a.row_perm, a.col_perm, a.m, a.level, a.byte_off, a.codes, a.scale,
                       a.zero, a.gc, a.opu, a.aborted);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

template <int LPG>
static int launch_gpack_l(sbits_ctx *ctx, const FusedPackLaunch &a)
{
    const int64_t chunks = a.cols / 8;
    if (chunks <= 512) return launch_gpack_g<LPG, 1, 4, 512>(ctx, a);
    if (chunks <= 1024) return launch_gpack_g<LPG, 2, 2, 512>(ctx, a);
    if (chunks <= 2048) return launch_gpack_g<LPG, 2, 2, 1024>(ctx, a);
    if (chunks <= 4096) return launch_gpack_g<LPG, 2, 2, 1024, 2>(ctx, a);
    return SBITS_ERR_BAD_SHAPE;
}

}  // namespace sbits

using namespace sbits;

// shapes the fused kernels take: 64- or 128-column blocks
// The route is chosen per class of matrices with equal column count.  Rows of up to FU_MAX_COLS
// elements are staged whole (weights and sensitivities) by gather_cost_kernel, wider ones (up to the plan's limit of 32768) by
// gather_cost_wide_kernel (fused_wide.hip) or, one matrix of few rows, by way of a reordered copy (few_wide_rows).  The surrogates take the first alone; the packing kernel stages weights only and
// takes every row length.
bool sbits_fused_shapes_ok(const sbits_plan *plan)
{
    if (plan->n != 64 && plan->n != 128) return false;
    return plan->max_cols <= FU_PACK_MAX_COLS;
}
// 32- and 256-column blocks: one pass that writes both copies
bool sbits_copies_shapes_ok(const sbits_plan *plan) { return plan->n == 32 || plan->n == 256; }
bool sbits_fused_all_staged(const sbits_plan *plan)
{
    return sbits_fused_shapes_ok(plan) && plan->max_cols <= FU_MAX_COLS;
}

static size_t octet_partial_bytes(const sbits_plan *plan)
{
    const size_t per_octet = (size_t)(plan->K > 2 ? plan->K : 2);     // the surrogates keep two sums per block
    return sbits_align_up((size_t)plan->N * (size_t)(plan->m / 8) * per_octet * 4, 256);
}
// One matrix of few wide rows, reordered into a copy in the workspace and scored there: eight rows of an octet one after the other, as
// gather_cost_wide_kernel takes them, are 25 us and more however few workgroups there are, the passes over such a copy 24 to 44.  Copy /
// one pass, 128-column blocks: 8 x 32768 at three candidates 28.9 us and 33.2, at nine 32.6 and 43.5; 128 x 32768 32.8 and 34.6, 36.5 and 43.8;
// 224 x 16512 29.4 and 27.4, 33.2 and 36.0; 224 x 24576 36.4 and 30.4, 45.3 and 38.3.  64 columns: two candidates 8 x 28672 27.4 and 32.3 (128
// columns 27.2 and 30.8, but 8 x 16512 25.0 and 25.6), nine 160 x 16512 38.4 and 36.6, 96 x 28672 40.3 and 44.3.  Two matrices of 8 x 16512: 41.2 and 29.4.
static bool few_wide_rows(const sbits_plan *plan, const sbits_plan::FusedClass &fc)
{
    if (!sbits_fused_shapes_ok(plan) || fc.cols <= FU_MAX_COLS || fc.n != 1 || plan->K < (plan->n == 64 ? 2 : 3)) return false;
    return plan->rows[plan->fused_members[fc.first]] * fc.cols <= (int64_t)4 << 20;
}

// octet partials: one float per (block, octet of the block, candidate); then room for the largest such copy (bf16, then fp32)
size_t sbits_fused_ws_bytes(const sbits_plan *plan)
{
    if (!sbits_copies_shapes_ok(plan) && !sbits_fused_shapes_ok(plan)) return 0;
    size_t copy = 0;
    for (const sbits_plan::FusedClass &fc : plan->fused_classes) {
        if (!few_wide_rows(plan, fc)) continue;
        const size_t el = (size_t)plan->rows[plan->fused_members[fc.first]] * (size_t)fc.cols;
        const size_t b = sbits_align_up(el * 2, 256) + sbits_align_up(el * 4, 256);
        if (b > copy) copy = b;
    }
    return octet_partial_bytes(plan) + copy;
}

// The cost and surrogate kernels rely on 16-bit register-half loads filling the other half with
// zeros (the device's target id says "sramecc+"); packing has instances that do not.  (That every source row starts on a 16-byte boundary,
// which the row loads need, is a rule of every entry point that takes matrices: checked there.)
bool sbits_fused_layout_ok(const sbits_plan *plan)
{
    return plan->ctx->d16_zero_fill;
}

// matrices grouped by column count: members and workgroup prefixes, class after class
void sbits_fused_tables(sbits_plan *plan)
{
    std::vector<int64_t> classes;
    for (int i = 0; i < plan->n_mats; ++i) {
        bool seen = false;
        for (int64_t c : classes) seen = seen || c == plan->cols[i];
        if (!seen) classes.push_back(plan->cols[i]);
    }
    for (int64_t c : classes) {
        sbits_plan::FusedClass fc;
        fc.cols = c;
        fc.first = (int)plan->fused_members.size();
        fc.pre_first = (int)plan->fused_pre.size();
        fc.n = 0;
        // octets per workgroup: FU_OPU, halved while the class would not even give every CU a few
        // workgroups (one decoder layer of a streamed model is such a plan)
        // (the last halving, to one octet, only while there is less than one per CU: 512 x 512 cost 18.7 -> 10.7 us, packing 8.4 -> 5.7)
        const int cus = sbits_cus(plan->ctx);
        int opu = FU_OPU;
        auto class_wgs = [&](int o) {
            int64_t t = 0;
            for (int i = 0; i < plan->n_mats; ++i)
                if (plan->cols[i] == c) t += (plan->rows[i] / 8 + o - 1) / o;
            return t;
        };
        while (opu > 1 && class_wgs(opu) < (opu > 2 ? 8 * cus : cus)) opu >>= 1;
        fc.opu = opu;
        int64_t t = 0;
        for (int i = 0; i < plan->n_mats; ++i) {
            if (plan->cols[i] != c) continue;
            plan->fused_members.push_back(i);
            plan->fused_pre.push_back((int)t);
            t += (plan->rows[i] / 8 + opu - 1) / opu;
            ++fc.n;
        }
        if (t > 0x7fffffff) { plan->fused_members.clear(); plan->fused_pre.clear(); plan->fused_classes.clear(); return; }
        plan->fused_pre.push_back((int)t);
        plan->fused_classes.push_back(fc);
    }
}

static int fused_classes(sbits_plan *plan, void *ws, const int **d_mem, const int **d_pre)
{
    if (plan->fused_classes.empty()) return SBITS_ERR_BAD_SHAPE;
    *d_mem = sbits_prefix_ptr(plan, ws, SLOT_FUSED_MEMBERS);
    *d_pre = sbits_prefix_ptr(plan, ws, SLOT_FUSED_WGS);
    return SBITS_OK;
}

// One launch per class of matrices with equal column count (equal LDS need, equal chunks per
// lane); the descriptor table is already in the workspace head.  w_re may be null, s_re is, except for 32- and 256-column blocks,
// where both are written.
int sbits_launch_fused_copies(int n, int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a);
int sbits_launch_fused_wide(int n, int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a);
int sbits_launch_gather_cost_all(sbits_plan *plan, const int32_t *row_perm, const int32_t *col_perm,
                                 void *w_re, float *s_re, float *cost, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    const bool copies = sbits_copies_shapes_ok(plan);
    if ((!copies && !sbits_fused_shapes_ok(plan)) || !sbits_fused_layout_ok(plan)) return SBITS_ERR_BAD_SHAPE;
    if (copies ? !w_re || !s_re : s_re != nullptr) return SBITS_ERR_INVALID_ARG;
    const int *d_mem, *d_pre;
    int rc0 = fused_classes(plan, ws, &d_mem, &d_pre);
    if (rc0) return rc0;
    FusedLaunch a;
    memset(&a, 0, sizeof a);
    a.descs = sbits_desc_ptr(ws);
    a.row_perm = row_perm;
    a.col_perm = col_perm;
    a.m = plan->m;
    a.w_re = static_cast<uint16_t *>(w_re);
    a.s_re = s_re;
    a.part = static_cast<float *>(sbits_scratch(plan, ws));
    for (const sbits_plan::FusedClass &fc : plan->fused_classes) {
        a.members = d_mem + fc.first;
        a.wg_start = d_pre + fc.pre_first;
        a.n_members = fc.n;
        a.total_wg = plan->fused_pre[fc.pre_first + fc.n];
        a.cols = fc.cols;
        a.opu = fc.opu;
        if (a.total_wg == 0 || (copies && fc.cols > FU_MAX_COLS) || few_wide_rows(plan, fc)) continue;
        const bool z0 = plan->bits[0] == 0;                     // a 0-bit candidate (the first of the list) has no grid
        sbits_fill_grid_consts(plan->bits + z0, plan->K - z0, &a.gc);
        a.kstride = plan->K;
        a.koff = 0;
        const int rc = copies ? sbits_launch_fused_copies(plan->n, plan->K, z0, ctx, a)
                     : fc.cols > FU_MAX_COLS ? sbits_launch_fused_wide(plan->n, plan->K, z0, ctx, a)
                     : plan->n == 64 ? launch_fused_l<8>(plan->K, z0, ctx, a) : launch_fused_l<16>(plan->K, z0, ctx, a);
        if (rc) return rc;
    }
    const int64_t NK = plan->N * plan->K;
    if (NK > 0) {
        hipLaunchKernelGGL(octet_finish_kernel, dim3((unsigned)((NK + 255) / 256)), dim3(256), 0, ctx->stream,
                           a.part, a.descs, plan->n_mats, NK, plan->K, plan->m / 8, cost);
        SBITS_HIP(ctx, hipGetLastError());
    }
    // matrices with rows too wide to stage (32- and 256-column blocks), or few of them: reordered first, then scored; their
    // rows of the table are written after the tree kernel above (which found nothing of theirs in part[])
    char *const room = static_cast<char *>(sbits_scratch(plan, ws)) + octet_partial_bytes(plan);
    for (const sbits_plan::FusedClass &fc : plan->fused_classes) {
        if (copies ? fc.cols <= FU_MAX_COLS : !few_wide_rows(plan, fc)) continue;
        for (int k = 0; k < fc.n; ++k) {
            const int i = plan->fused_members[fc.first + k];
            const MatDesc &d = plan->descs[i];
            void *w_i = w_re ? static_cast<void *>(static_cast<uint16_t *>(w_re) + d.elem_off) : static_cast<void *>(room);
            float *s_i = copies ? s_re + d.elem_off : reinterpret_cast<float *>(room + sbits_align_up((size_t)plan->rows[i] * (size_t)plan->cols[i] * 2, 256));
            int rc = sbits_launch_gather(ctx, d.w, d.s, plan->rows[i], plan->cols[i], d.ld_w, d.ld_s, row_perm + d.row_off,
                                         col_perm + d.col_off, w_i, s_i);
            if (rc) return rc;
            rc = sbits_launch_cost(ctx, w_i, s_i, plan->rows[i], plan->cols[i], plan->m, plan->n, plan->bits, plan->K,
                                   cost + d.block_base * plan->K);
            if (rc) return rc;
        }
    }
    return SBITS_OK;
}

// the packing stage on the original weights, one launch per class
int sbits_launch_gather_pack_all(sbits_plan *plan, const int32_t *row_perm, const int32_t *col_perm,
                                 const uint8_t *level, const int64_t *byte_off, uint8_t *codes, float *scale,
                                 float *zero, void *ws, const unsigned *aborted)
{
    sbits_ctx *ctx = plan->ctx;
    if (!sbits_fused_shapes_ok(plan)) return SBITS_ERR_BAD_SHAPE;
    const int *d_mem, *d_pre;
    int rc0 = fused_classes(plan, ws, &d_mem, &d_pre);
    if (rc0) return rc0;
    FusedPackLaunch a;
    memset(&a, 0, sizeof a);
    sbits_fill_grid_consts(plan->bits, plan->K, &a.gc);
    a.descs = sbits_desc_ptr(ws);
    a.row_perm = row_perm;
    a.col_perm = col_perm;
    a.m = plan->m;
    a.level = level; a.byte_off = byte_off; a.codes = codes; a.scale = scale; a.zero = zero;
    a.wide = plan->bits[plan->K - 1] > 4;
    a.mask = !ctx->d16_zero_fill;
    a.aborted = aborted;
    for (const sbits_plan::FusedClass &fc : plan->fused_classes) {
        a.members = d_mem + fc.first;
        a.wg_start = d_pre + fc.pre_first;
        a.n_members = fc.n;
        a.total_wg = plan->fused_pre[fc.pre_first + fc.n];
        a.cols = fc.cols;
        a.opu = fc.opu;
        if (a.total_wg == 0) continue;
        const int rc = plan->n == 64 ? launch_gpack_l<8>(ctx, a) : launch_gpack_l<16>(ctx, a);
        if (rc) return rc;
    }
    return SBITS_OK;
}

// dynamic-sensitivity surrogates of all matrices: the one-pass kernel in its second mode, then the
// tree over the octets with the 2^-bits factor of s_down
int sbits_launch_surrogates_all(sbits_plan *plan, const int32_t *row_perm, const int32_t *col_perm,
                                const uint8_t *level, float *s_up, float *s_down, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    if (!sbits_fused_all_staged(plan) || !sbits_fused_layout_ok(plan)) return SBITS_ERR_BAD_SHAPE;
    const int *d_mem, *d_pre;
    int rc0 = fused_classes(plan, ws, &d_mem, &d_pre);
    if (rc0) return rc0;
    FusedLaunch a;
    memset(&a, 0, sizeof a);
    sbits_fill_grid_consts(plan->bits, plan->K, &a.gc);
    a.descs = sbits_desc_ptr(ws);
    a.row_perm = row_perm;
    a.col_perm = col_perm;
    a.m = plan->m;
    a.w_re = nullptr;
    a.part = static_cast<float *>(sbits_scratch(plan, ws));
    a.level = level;
    a.kstride = 2;
    a.koff = 0;
    for (const sbits_plan::FusedClass &fc : plan->fused_classes) {
        a.members = d_mem + fc.first;
        a.wg_start = d_pre + fc.pre_first;
        a.n_members = fc.n;
        a.total_wg = plan->fused_pre[fc.pre_first + fc.n];
        a.cols = fc.cols;
        a.opu = fc.opu;
        if (a.total_wg == 0) continue;
        const int rc = plan->n == 64 ? launch_surrogates_l<8>(ctx, a) : launch_surrogates_l<16>(ctx, a);
        if (rc) return rc;
    }
    if (plan->N > 0) {
        hipLaunchKernelGGL(surrogate_finish_kernel, dim3((unsigned)((2 * plan->N + 255) / 256)), dim3(256), 0,
                           ctx->stream, a.part, a.descs, plan->n_mats, plan->N, plan->m / 8, level, a.gc, s_up, s_down);
        SBITS_HIP(ctx, hipGetLastError());
    }
    return SBITS_OK;
}
