// The stored matrix back as numbers (paper Sec. 5.3: codes with one bitwidth per tile, scale and
// zero per block row): What[i][j] = fmaf(code, scale, zero), in the reordered coordinates the stream
// was packed in, as fp32 (exact: this is the format's definition of the stored value) or rounded to
// bf16 (nearest even).  A utility beside the inference product: for evaluating a quantized model
// with ordinary dense kernels, and for checking.  Write-bound: c / 8 bytes read, 4 (or 2) written
// per weight.
//
// One lane per 16 bytes of output (8 columns in bf16, 4 in fp32) of four rows of one block row: the block's level and
// place in the stream are looked up once for the four, and every store of a wave is 1 KiB of consecutive bytes.
// Codes 0 .. 3 of a lane (4 c <= 32 bits, whatever c is) come out of two aligned dwords with one funnel
// shift, codes 4 .. 7 with another, so lanes on blocks of different bitwidths run the same instructions.
// What bounds it: the writes.  8192 x 28672 of {2,3,4} bits, three outputs written in turn: to bf16 229 us with a lane
// per run of 8 codes (lookups and 64-bit shifts per run) -> 117 us (4.9 TB/s read and written; 83 us where the output fits the
// last-level cache), to fp32 305 -> 204 us.  One wave per workgroup and four rows: 8 and 16 rows take 124 and 132 us,
// workgroups of 256 threads 118 us there and 39 us instead of 24 on 14336 x 4096 with 32-column blocks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sbits_internal.hpp"

namespace sbits {

constexpr int DQ_ROWS = 4;                   // rows of a workgroup (block rows are a multiple of 8)

struct DequantArgs {
    const uint8_t *codes;
    const float *scale, *zero;
    const uint8_t *level;
    const int64_t *byte_off;
    void *out;
    int64_t block_base, ld_out;
    int R, C, m, n_log2, nbc;
    int bits[MAX_CAND];
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef f32x4_t __attribute__((aligned(4))) f32x4_a4_t;       // (scale and zero are aligned to their elements only)

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)      // nearest even
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

template <bool BF16>
__global__ __launch_bounds__(64)
void dequant_kernel(DequantArgs a)
{
    constexpr int V = BF16 ? 8 : 4;                           // columns per lane
    const int j = (int)(blockIdx.x * 64 + threadIdx.x) * V;
    if (j >= a.C) return;
    const int i0 = (int)blockIdx.y * DQ_ROWS;                 // first row; all of them in one block row
    const int I = i0 / a.m, r0 = i0 - I * a.m;
    const int J = j >> a.n_log2, cin = j - (J << a.n_log2);
    const int64_t blk = a.block_base + (int64_t)I * a.nbc + J;
    const int lv = a.level[blk];
    int bits = a.bits[0];
#pragma unroll
    for (int k = 1; k < MAX_CAND; ++k) bits = lv == k ? a.bits[k] : bits;
    // the block's stream (at most 1024 x 512 codes of 8 bits: bit offsets fit 32 bits)
    const uint32_t c = (uint32_t)bits;
    const uint8_t *base = a.codes + a.byte_off[blk];
    const uint32_t end = (uint32_t)((a.m << a.n_log2) >> 3) * c - 4u;                      // its last dword
    const uint32_t pitch = c << a.n_log2;                     // bits of one row's codes
    const uint32_t off = (uint32_t)r0 * pitch + (uint32_t)cin * c;
    const float *ps = a.scale + blk * a.m + r0, *pz = a.zero + blk * a.m + r0;
    typedef const __attribute__((address_space(1))) uint32_t gu32;
    uint32_t w[DQ_ROWS][V == 8 ? 3 : 2];
    const f32x4_t sc = *(const f32x4_a4_t *)ps, ze = *(const f32x4_a4_t *)pz;
#pragma unroll
    for (int u = 0; u < DQ_ROWS; ++u) {
        const uint32_t q = (off + (uint32_t)u * pitch) >> 5 << 2;
        w[u][0] = w[u][1] = 0u;
        if constexpr (V == 8) w[u][2] = 0u;
        if (bits) {                                       // (a pruned block has no codes: its value is zero[] = 0)
            w[u][0] = *(gu32 *)(base + q);
            w[u][1] = *(gu32 *)(base + min(q + 4u, end)); // (past the block's end: not needed, not read)
            if constexpr (V == 8) w[u][2] = *(gu32 *)(base + min(q + 8u, end));
        }
    }
#pragma unroll
    for (int u = 0; u < DQ_ROWS; ++u) {
        const uint32_t sh = (off + (uint32_t)u * pitch) & 31u;
        const uint32_t lo = __builtin_amdgcn_alignbit(w[u][1], w[u][0], sh);
        float v[V];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaf((float)__builtin_amdgcn_ubfe(lo, (uint32_t)e * c, c), sc[u], ze[u]);
        const int64_t at = (int64_t)(i0 + u) * a.ld_out + j;
        if constexpr (BF16) {
            const uint32_t sh4 = sh + 4u * c;             // sh <= 24 here
            const bool far = sh4 >= 32u;
            const uint32_t hi = __builtin_amdgcn_alignbit(far ? w[u][2] : w[u][1], far ? w[u][1] : w[u][0], sh4 & 31u);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 + e] = fmaf((float)__builtin_amdgcn_ubfe(hi, (uint32_t)e * c, c), sc[u], ze[u]);
            const u32x4_t t = {bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]), bf16_pair(v[4], v[5]), bf16_pair(v[6], v[7])};
            __builtin_nontemporal_store(t, (__attribute__((address_space(1))) u32x4_t *)(static_cast<uint16_t *>(a.out) + at));
        } else {
            const f32x4_t t = {v[0], v[1], v[2], v[3]};
            __builtin_nontemporal_store(t, (__attribute__((address_space(1))) f32x4_t *)(static_cast<float *>(a.out) + at));
        }
    }
}

}  // namespace sbits

using namespace sbits;

int sbits_launch_dequant(sbits_plan *plan, int mat, const uint8_t *level, const int64_t *byte_off,
                         const uint8_t *codes, const float *scale, const float *zero, void *out, int64_t ld_out,
                         int out_bf16)
{
    sbits_ctx *ctx = plan->ctx;
    DequantArgs a;
    a.codes = codes; a.scale = scale; a.zero = zero; a.level = level; a.byte_off = byte_off;
    a.out = out; a.block_base = plan->base[mat]; a.ld_out = ld_out;
    a.R = (int)plan->rows[mat]; a.C = (int)plan->cols[mat]; a.m = plan->m; a.nbc = a.C / plan->n;
    a.n_log2 = 0;
    while ((1 << a.n_log2) < plan->n) ++a.n_log2;
    for (int c = 0; c < sbits::MAX_CAND; ++c) a.bits[c] = c < plan->K ? plan->bits[c] : plan->bits[plan->K - 1];
    const int v = out_bf16 ? 8 : 4;                           // columns per lane
    const unsigned gx = (unsigned)((a.C / v + 63) / 64);
    const dim3 grid(gx, (unsigned)(a.R / DQ_ROWS));
    if (out_bf16) hipLaunchKernelGGL(dequant_kernel<true>, grid, dim3(64), 0, ctx->stream, a);
    else hipLaunchKernelGGL(dequant_kernel<false>, grid, dim3(64), 0, ctx->stream, a);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}
