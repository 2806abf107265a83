// Product of a small batch of activations with the stored mixed-precision weights (paper Sec. 5.3
// "Inference Kernel": dequantization fused into the matrix product, at the granularity of the
// precision blocks, one bitwidth per tile, no divergence inside a wave):
//
//     y[b][i] = sum_j What[i][j] * x[b][j],      What[i][j] = q[i][j] * scale[i][J] + zero[i][J]
//
// for one matrix of the plan, read straight from the packed stream of sbits_pack (blocks in global
// order, rows of a block one after the other, LSB-first codes, scale / zero per block row).
//
// The sum over a block row's n columns splits as  scale * (sum_j q x) + zero * (sum_j x):
// the matrix cores multiply the integer codes (exact in bf16) with x, a second product with
// an all-ones operand gives sum_j x in the same register layout, and two fp32 FMAs per output and
// block apply the row's scale and zero.  For bitwidths below 8 the codes enter as bf16 128 + q
// (the code OR-ed into the mantissa of 128.0: no integer-to-float conversion), and the offset is
// folded into the zero term: zero' = zero - 128 * scale.
//
// Mapping (v_mfma_f32_16x16x32_bf16: A = x, 16 batch rows; B = What^T, 16 output channels; K = 32):
//   lane l supplies channel i = l % 16 and the K-quarter g = l / 16 of a block row: its n / 4 codes
//   are n * c / 32 consecutive bytes of the stream; the wave's 16 rows x n codes are one contiguous
//   run.  A workgroup covers 1, 2 or 4 row groups of 32 rows (2 channel tiles each; by the size of the
//   product) x 16 block columns (4 waves per row group, 4 blocks per wave, two or three of them in flight
//   in a ring of register slots); the x slice of those columns sits in LDS.  Block columns beyond the first 16
//   go to further workgroups (grid.y), whose partial sums a second kernel adds in a fixed order.
//   Workgroups of 4 row groups leave no room for a second one on the CU, so nothing ran while one started
//   or ended: with 2 of 512 threads 9344 x 9344 at 5 rows took 18.5 us instead of 22.2.  Codes come by two
//   loads whatever the bitwidth (load_quarter): with one path per bitwidth the ring was copied at the paths'
//   end, behind a wait for it, 5824 x 6144 at 23 rows 17.7 -> 15.6 us; 64-column blocks, before two bytes
//   at a time, 960 x 23872 at 13 rows 31.8 -> 16.5.
// More than 32 batch rows, and products of up to 64 where few_rows says so (most of up to 16), take the kernels further down.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sbits_internal.hpp"

namespace sbits {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4v_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

constexpr int MG_JL = 4;                 // waves per row group, each on its own block columns
constexpr int MG_NBLK = 4;               // blocks per wave
constexpr int MG_SPAN = MG_JL * MG_NBLK; // block columns per workgroup

struct MpArgs {
    const uint8_t *codes;
    const float *scale, *zero;
    const uint8_t *level;
    const int64_t *byte_off;
    const uint16_t *x;                   // bf16 [batch][ld_x]
    float *out;                          // y [batch][R] (n_split == 1) or partials [n_split][batch][R]
    int64_t block_base, ld_x;
    int R, C, m, nbc, batch, n_split;
    int bits[MAX_CAND];
};

__device__ __forceinline__ bf16x8_t as_bf16x8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    u32x4_t v;
    v.x = a; v.y = b; v.z = c; v.w = d;
    return __builtin_bit_cast(bf16x8_t, v);
}

// code e (0 .. 8 * words - 1) of the lane's LSB-first stream, C bits
template <int C>
__device__ __forceinline__ uint32_t code_at(const uint32_t (&r)[8], int e)
{
    const int bit = e * C, idx = bit >> 5, sh = bit & 31;
    uint32_t v = r[idx] >> sh;
    if (sh + C > 32) v |= r[idx + 1] << (32 - sh);
    return v & ((1u << C) - 1u);
}

// Operands of the products of more than 32 rows, two codes in three instructions whatever the bitwidth c <= 7: field
// extraction, spread to the two halves, mask and exponent.  c <= 5: B = 1 + q / 2^c (the code at the top of the
// mantissa: the offset taken out again is no larger than the codes' range), c = 6, 7: B = 128 + q, c = 8: B = q.
// the exponents of a pair (in a vector register) and the codes' places (in a scalar one): held in registers the last two
// operations are one instruction, which takes no literals
template <int C> struct PairConst {
    static constexpr uint32_t one = C <= 5 ? 0x3f803f80u : 0x43004300u;
    static constexpr uint32_t field = C <= 5 ? ((1u << C) - 1u) << (7 - C) : (1u << C) - 1u;
};
template <int C>
__device__ __forceinline__ uint32_t code_pair(const uint32_t *r, int e, uint32_t one, uint32_t mask)   // codes e, e + 1 (e even) as two bf16
{
    if constexpr (C == 8) {
        const uint32_t w = r[e >> 2];
        const uint32_t f0 = __float_as_uint((float)((w >> (8 * (e & 3))) & 255u)), f1 = __float_as_uint((float)((w >> (8 * (e & 3) + 8)) & 255u));
        return __builtin_amdgcn_perm(f1, f0, 0x07060302u);
    } else {
        const int bit = e * C, idx = bit >> 5, sh = bit & 31;
        if constexpr (C == 2)                                 // (the byte is selected by the multiplication; its two pairs differ in the factor)
            return (__umul24((r[idx] >> (sh & 24)) & 255u, sh & 4 ? (1u << 1) + (1u << 15) : (1u << 5) + (1u << 19)) & mask) | one;
        const uint32_t x = sh + 2 * C <= 32 ? __builtin_amdgcn_ubfe(r[idx], sh, 2 * C)
                                            : __builtin_amdgcn_alignbit(r[idx + 1], r[idx], sh) & ((1u << (2 * C)) - 1u);
        // C <= 5: the copies of the two codes do not overlap where the mask looks, nor carry into it
        const uint32_t y = C <= 5 ? __umul24(x, (1u << (7 - C)) + (1u << (23 - 2 * C))) : x | x << (16 - C);
        return (y & mask) | one;
    }
}

// the block's scale and zero as they apply to sum B x and sum x
template <int C>
__device__ __forceinline__ void term_factors(float sc, float ze, float &f, float &z)
{
    f = C <= 5 ? sc * (float)(1 << C) : sc;
    z = C <= 5 ? fmaf(-(float)(1 << C), sc, ze) : C < 8 ? fmaf(-128.0f, sc, ze) : ze;
}

// B operand of step `st`: the lane's codes 8 * st .. 8 * st + 7 as bf16, in stream order.
// C < 8: 128 + q (the code in the mantissa of 128.0);  C == 8: q itself (converted).  FINE: as code_pair().
template <int C, bool FINE>
__device__ __forceinline__ bf16x8_t operand(const uint32_t (&r)[8], int st)
{
    uint32_t w[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if constexpr (FINE) {
            w[p] = code_pair<C>(r, 8 * st + 2 * p, PairConst<C>::one, PairConst<C>::field * 0x10001u);
            continue;
        }
        const uint32_t q0 = code_at<C>(r, 8 * st + 2 * p), q1 = code_at<C>(r, 8 * st + 2 * p + 1);
        if constexpr (C < 8) {
            w[p] = 0x43004300u | q0 | (q1 << 16);
        } else {
            const uint32_t f0 = __float_as_uint((float)q0), f1 = __float_as_uint((float)q1);   // <= 8 significant bits
            w[p] = (f0 >> 16) | (f1 & 0xffff0000u);
        }
    }
    return as_bf16x8(w[0], w[1], w[2], w[3]);
}

// ---- pair order (bitwidths 1, 2, 4): a 32-bit word holds two codes 16 bits apart, so one AND-OR
// turns  (w >> s) & mask  into the bf16 pair (128 + q_a, 128 + q_b) with b - a = 16 / C codes.
// The operand then holds the lane's codes in the order a0, b0, a1, b1, ...; x is put into the
// same order with byte permutes (x_operand; shared by both channel tiles).
//   C = 4: step st, pair p: codes (8 st + p,        8 st + p + 4)     word st,      shift 4 p
//   C = 2: step st, pair p: codes (16 d + 4 h + p,  ... + 8)          word d,       shift 2 (4 h + p),  st = 2 d + h
//   C = 1: step st, pair p: codes (4 st + p,        4 st + p + 16)    word 0,       shift 4 st + p      (32 codes per lane only)
template <int C, int KL>
struct PairOrder {
    static constexpr bool value = C == 4 || C == 2 || (C == 1 && KL == 32);
};

template <int C, bool FINE>
__device__ __forceinline__ bf16x8_t operand_pairs(const uint32_t (&r)[8], int st)
{
    uint32_t w[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if constexpr (FINE) {                                 // (the codes to the mantissa's top)
            const uint32_t word = C == 4 ? r[st] : C == 2 ? r[st >> 1] : r[0];
            const int sh = (C == 4 ? 4 * p : C == 2 ? 2 * (4 * (st & 1) + p) : 4 * st + p) - (7 - C);
            w[p] = ((sh < 0 ? word << -sh : word >> (sh < 0 ? 0 : sh)) & PairConst<C>::field * 0x10001u) | PairConst<C>::one;
        } else if constexpr (C == 4) w[p] = ((r[st] >> (4 * p)) & 0x000f000fu) | 0x43004300u;
        else if constexpr (C == 2) w[p] = ((r[st >> 1] >> (2 * (4 * (st & 1) + p))) & 0x00030003u) | 0x43004300u;
        else w[p] = ((r[0] >> (4 * st + p)) & 0x00010001u) | 0x43004300u;
    }
    return as_bf16x8(w[0], w[1], w[2], w[3]);
}

// The lane's codes of one block row quarter, `at` bytes into the block, as raw as they come: always the same two loads
// into the same registers, whatever the bitwidth (a choice by bitwidth ends in copies, and a copy waits for its load).
// They go through a descriptor of exactly the block's bytes: what lies past its end reads as zero and is not fetched.
// 128 columns: up to 8 dwords from a multiple of 4 bytes on.  64 columns: up to 16 bytes from a multiple of 2 on, so the
// 5 aligned dwords around them, which align_quarter() shifts into place.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
template <int N_COLS>
struct Quarter { uint32_t r[N_COLS == 128 ? 8 : 5]; };
template <int N_COLS>
__device__ __forceinline__ void load_quarter(rsrc_t rs, uint32_t at, Quarter<N_COLS> &o)
{
    const int off = (int)(N_COLS == 128 ? at : at & ~3u);
    const u32x4_t v = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    o.r[0] = v.x; o.r[1] = v.y; o.r[2] = v.z; o.r[3] = v.w;
    if constexpr (N_COLS == 128) {
        const u32x4_t h = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0));
        o.r[4] = h.x; o.r[5] = h.y; o.r[6] = h.z; o.r[7] = h.w;
    } else {
        o.r[4] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 16, 0, 0);
    }
}
template <int N_COLS>
__device__ __forceinline__ void align_quarter(const Quarter<N_COLS> &q, uint32_t at, uint32_t (&r)[N_COLS / 16])
{
#pragma unroll
    for (int i = 0; i < N_COLS / 16; ++i)
        r[i] = N_COLS == 128 ? q.r[i] : __builtin_amdgcn_alignbit(q.r[i + 1 < 5 ? i + 1 : 4], q.r[i], (at & 2u) * 8u);
}

// x operand of step st, read from the lane's 2 * KL bytes of the staged slice (natural order in LDS).
// Stream order: the step's 16 bytes as they are.  Pair order of bitwidth C: the two elements of pair
// p sit in the same half of two words 16 / C codes apart, fetched as two 8-byte reads and merged
// with byte permutes.
template <int C, bool PAIRS>
__device__ __forceinline__ bf16x8_t x_operand(const unsigned char *xl, int st)
{
    if constexpr (!PAIRS) {
        return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(xl + 16 * st));
    } else {
        int ea, gap;                                  // first element of pair 0; distance to its partner
        if constexpr (C == 4) { ea = 8 * st; gap = 4; }
        else if constexpr (C == 2) { ea = 16 * (st >> 1) + 4 * (st & 1); gap = 8; }
        else { ea = 4 * st; gap = 16; }
        // pairs p = 0..3 use elements ea + p and ea + p + gap: words (ea >> 1) + {0, 1} and the same + gap / 2
        const u32x2_t wa = *reinterpret_cast<const u32x2_t *>(xl + 2 * ea);
        const u32x2_t wb = *reinterpret_cast<const u32x2_t *>(xl + 2 * (ea + gap));
        uint32_t w[4];
        w[0] = __builtin_amdgcn_perm(wb.x, wa.x, 0x05040100u);
        w[1] = __builtin_amdgcn_perm(wb.x, wa.x, 0x07060302u);
        w[2] = __builtin_amdgcn_perm(wb.y, wa.y, 0x05040100u);
        w[3] = __builtin_amdgcn_perm(wb.y, wa.y, 0x07060302u);
        return as_bf16x8(w[0], w[1], w[2], w[3]);
    }
}

// One block: loads were issued before (cw, sc, ze); multiply and add into acc.
template <int C, int N_COLS, int NB, bool FINE>
__device__ __forceinline__ void block_product(const uint32_t (&cw)[2][8], const float (&sc)[2], const float (&ze)[2],
                                              const unsigned char *const (&xl)[NB], f32x4v_t (&acc)[2][NB])
{
    constexpr int STEPS = N_COLS / 32;
    constexpr bool PAIRS = PairOrder<C, N_COLS / 4>::value;
    const bf16x8_t ones = as_bf16x8(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    f32x4v_t d[2][NB], d1[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        d1[nb] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};
        d[0][nb] = d1[nb];
        d[1][nb] = d1[nb];
    }
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        bf16x8_t b0, b1;
        if constexpr (PAIRS) { b0 = operand_pairs<C, FINE>(cw[0], st); b1 = operand_pairs<C, FINE>(cw[1], st); }
        else { b0 = operand<C, FINE>(cw[0], st); b1 = operand<C, FINE>(cw[1], st); }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const bf16x8_t xa = x_operand<C, PAIRS>(xl[nb], st);
            d[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, b0, d[0][nb], 0, 0, 0);
            d[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, b1, d[1][nb], 0, 0, 0);
            d1[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, ones, d1[nb], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        float f = sc[t], zz = C < 8 ? fmaf(-128.0f, sc[t], ze[t]) : ze[t];
        if constexpr (FINE) term_factors<C>(sc[t], ze[t], f, zz);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[t][nb][r] = fmaf(f, d[t][nb][r], fmaf(zz, d1[nb][r], acc[t][nb][r]));
    }
}

// Codes, scales and zeros of block T of a wave -> register slot S; the same number of load
// instructions whatever the block.  c = 0: a block column beyond the matrix, or a pruned block (0 bits:
// an empty descriptor, nothing fetched; the clamped block's scales).  (A macro: through a function the slots end up in
// scratch memory.)
#define MG_REQUEST(T, S)                                                                                          \
    do {                                                                                                          \
        const uint64_t at_ = ((uint64_t)off_hi[T] << 32) | off_lo[T];                                             \
        const rsrc_t rs_ = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.codes) + at_, 0,             \
            (int)((uint32_t)(a.m * (N_COLS / 8)) * (uint32_t)cbits[T]), 0x00027000);                              \
        const float *ps_ = a.scale + blk[T] * a.m + rin, *pz_ = a.zero + blk[T] * a.m + rin;                      \
        _Pragma("unroll") for (int tl = 0; tl < 2; ++tl) {                                                        \
            sc[S][tl] = ps_[16 * tl + li];                                                                        \
            ze[S][tl] = pz_[16 * tl + li];                                                                        \
            load_quarter<N_COLS>(rs_, (lane_units + (uint32_t)(tl * 16 * (N_COLS / 8))) * (uint32_t)cbits[T], cq[S][tl]); \
        }                                                                                                         \
    } while (0)

template <int N_COLS, int NB, int RG, bool FINE>
__global__ __launch_bounds__((64 * MG_JL * RG), 4)
void mp_gemm_kernel(MpArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int KL = N_COLS / 4, THREADS = 64 * MG_JL * RG;
    constexpr int SLICE = MG_SPAN * N_COLS;                    // x columns per workgroup
    constexpr int PITCH = SLICE * 2 + 16;                      // bytes per batch row in LDS (+16: spreads the rows over the banks)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: the bookkeeping below stays scalar
    const int rg = wave & (RG - 1), jl = wave / RG;
    const int li = lane & 15, g = lane >> 4;
    const int col0 = blockIdx.y * SLICE;                       // first x column of the slice
    const int J0 = blockIdx.y * MG_SPAN;

    // ---- this wave's blocks: all metadata loads first (they head the longest dependency chain);
    // a block column beyond the matrix reads the last one's metadata and is skipped later
    const int row0 = blockIdx.x * (RG * 32) + rg * 32;      // first of the wave's 32 rows
    const bool rows_ok = row0 < a.R;                           // (R is a multiple of 32)
    const int I = rows_ok ? row0 / a.m : 0, rin = rows_ok ? row0 - I * a.m : 0;
    // PF blocks of codes are in flight at a time (a ring of PF register slots, refilled after each
    // block): three with one batch tile (measured: 15.0 us against 15.3 with two and 16.3 with all four
    // requested at once, whose first block then arrives late), two with two batch tiles (registers)
    constexpr int PF = NB == 1 ? 3 : 2;
    int cbits[MG_NBLK];
    Quarter<N_COLS> cq[PF][2];
    float sc[PF][2], ze[PF][2];
    int64_t blk[MG_NBLK];
    uint32_t lvl_v[MG_NBLK];
    int64_t boff_v[MG_NBLK];
#pragma unroll
    for (int t = 0; t < MG_NBLK; ++t) {
        const int J = J0 + jl + MG_JL * t;
        blk[t] = a.block_base + (int64_t)I * a.nbc + (J < a.nbc ? J : a.nbc - 1);
        lvl_v[t] = a.level[blk[t]];
        boff_v[t] = a.byte_off[blk[t]];
    }
    // ---- x slice: requested together with the metadata (rows beyond the batch and columns beyond C read
    // as zero) and in LDS by the time the metadata has arrived
    constexpr int XCH = 16 * NB * (SLICE / 8) / THREADS;    // 16-byte pieces per thread
    static_assert(16 * NB * (SLICE / 8) % THREADS == 0, "whole pieces per thread");
    u32x4_t xs[XCH];
#pragma unroll
    for (int i = 0; i < XCH; ++i) {
        const int q = tid + i * THREADS;
        const int b = q / (SLICE / 8), ch = q - b * (SLICE / 8);
        const int bc = b < a.batch ? b : a.batch - 1;                               // in bounds; zeroed below
        const int cc = col0 + ch * 8 < a.C ? col0 + ch * 8 : 0;
        xs[i] = *(const __attribute__((address_space(1))) u32x4_t *)(a.x + (int64_t)bc * a.ld_x + cc);
    }

#pragma unroll
    for (int i = 0; i < XCH; ++i) {
        const int q = tid + i * THREADS;
        const int b = q / (SLICE / 8), ch = q - b * (SLICE / 8);
        const bool ok = b < a.batch && col0 + ch * 8 < a.C;
        u32x4_t v = xs[i];
        v.x = ok ? v.x : 0u; v.y = ok ? v.y : 0u; v.z = ok ? v.z : 0u; v.w = ok ? v.w : 0u;
        *reinterpret_cast<u32x4_t *>(smem + (size_t)b * PITCH + ch * 16) = v;
    }
    // (no global load is in flight here but the metadata: the codes are requested after the barrier)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the x slice is in LDS
    const uint32_t lane_units = (uint32_t)((rin + li) * (N_COLS / 8) + g * (KL / 8));   // x c = the lane's byte offset in the block
    // the blocks' bitwidths and stream offsets as scalars
    uint32_t off_lo[MG_NBLK], off_hi[MG_NBLK];
#pragma unroll
    for (int t = 0; t < MG_NBLK; ++t) {
        const int J = J0 + jl + MG_JL * t;
        const int lv = __builtin_amdgcn_readfirstlane((int)lvl_v[t]);
        int c = a.bits[0];
#pragma unroll
        for (int k = 1; k < MAX_CAND; ++k) c = lv == k ? a.bits[k] : c;
        cbits[t] = (rows_ok && J < a.nbc) ? c : 0;
        off_lo[t] = __builtin_amdgcn_readfirstlane((uint32_t)boff_v[t]);
        off_hi[t] = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)boff_v[t] >> 32));
    }
#pragma unroll
    for (int t = 0; t < PF; ++t) MG_REQUEST(t, t);

    f32x4v_t acc[2][NB];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[t][nb] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};

#pragma unroll
    for (int t = 0; t < MG_NBLK; ++t) {
        const int c = cbits[t];
        const int Jl = jl + MG_JL * t;                         // block column inside the slice
        const unsigned char *xa[NB];                           // the lane's x values of this block column (LDS, natural order)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            xa[nb] = smem + (size_t)(16 * nb + li) * PITCH + (size_t)(Jl * N_COLS + g * KL) * 2;
        uint32_t cw[2][8];
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
            uint32_t w[N_COLS / 16];
            align_quarter<N_COLS>(cq[t % PF][tl], (lane_units + (uint32_t)(tl * 16 * (N_COLS / 8))) * (uint32_t)c, w);
#pragma unroll
            for (int i = 0; i < N_COLS / 16; ++i) cw[tl][i] = w[i];
        }
        if (c != 0) switch (c) {                               // (0: no such block column, or a pruned block)
        case 1: block_product<1, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 2: block_product<2, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 3: block_product<3, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 4: block_product<4, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 5: block_product<5, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 6: block_product<6, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        case 7: block_product<7, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        default: block_product<8, N_COLS, NB, FINE>(cw, sc[t % PF], ze[t % PF], xa, acc); break;
        }
        if (t + PF < MG_NBLK) MG_REQUEST((t + PF) % MG_NBLK, t % PF);   // the slot is free again
    }

    // ---- the four waves of a row group add up (fixed order), wave jl = 0 stores
    __syncthreads();                                           // every wave is done with the x slice
    float *red = reinterpret_cast<float *>(smem);              // [wave][tile][nb][r][lane]
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[(((wave * 2 + t) * NB + nb) * 4 + r) * 64 + lane] = acc[t][nb][r];
    __syncthreads();
    if (jl != 0 || !rows_ok) return;
    float *dst = a.out + (int64_t)blockIdx.y * a.batch * a.R;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float v = acc[t][nb][r];
#pragma unroll
                for (int j = 1; j < MG_JL; ++j)
                    v = v + red[((((rg + RG * j) * 2 + t) * NB + nb) * 4 + r) * 64 + lane];
                const int b = 16 * nb + 4 * g + r;             // D layout: row 4 * (lane / 16) + r, column lane % 16
                if (b < a.batch) dst[(int64_t)b * a.R + row0 + 16 * t + li] = v;
            }
}

#define MP_SWITCH(c, F)                                                                                           \
    switch (c) {                                                                                                  \
    case 0: break;                                                                                                \
    case 1: F(1); break;                                                                                          \
    case 2: F(2); break;                                                                                          \
    case 3: F(3); break;                                                                                          \
    case 4: F(4); break;                                                                                          \
    case 5: F(5); break;                                                                                          \
    case 6: F(6); break;                                                                                          \
    case 7: F(7); break;                                                                                          \
    default: F(8); break;                                                                                         \
    }

// ================================================================ few batch rows
// Few rows of x are small next to the codes, so nothing is staged and no columns are split off: a workgroup takes 32
// channels, 16 rows of x and all columns, its 8 or 16 waves every 8th or 16th block column each, codes of two blocks in flight,
// and one exchange through LDS at the end.  Against the first kernel this takes the second launch, the partial sums in memory
// and the wait for x out, and a small matrix has more CUs; the price is x read once per 32 channels, and codes once per 16 rows.
// Products as there, in its column order; a wave of 8 keeps two sums, so that there are the same sixteen partial sums either way.
// Up to 4 rows the operands of x come straight from the caches.  With more, a lane's operand is 16 bytes of a row of its own:
// 64 lanes, 64 lines, and the L1 takes a line a clock.  There whole rows are read (16 lanes 256 bytes) and change lanes in LDS,
// private to the wave: 8192 x 8192 at 16 rows 15.7 -> 12.6 us.  Latency bounds it: level and offset, then codes, then
// the exchange; with several turns, vector issue (unpacking) and L2.
// 1024 x 4096, bitwidths 1 .. 4, one row: 11.3 -> 5.8 us; 4096 x 4096, 4 bits: 11.2 -> 5.9.  17 .. 32 rows, which all took
// the first kernel before: 1984 x 3328 at 26 rows 16.1 -> 8.2 us, 2112 x 1856 in 64-column blocks at 23 rows 14.9 -> 6.2.

// x operand of step st from the lane's KL values in registers: natural or, for the bitwidths of PairOrder, pair order
template <int C, int KL>
__device__ __forceinline__ bf16x8_t x_held(const u32x4_t (&x)[KL / 8], int st)
{
    if constexpr (!PairOrder<C, KL>::value) {
        return __builtin_bit_cast(bf16x8_t, x[st]);
    } else {
        const int ea = C == 4 ? 8 * st : C == 2 ? 16 * (st >> 1) + 4 * (st & 1) : 4 * st, eb = ea + 16 / C;   // (multiples of 4)
        auto word = [&](int e, int k) { return x[e >> 3][((e & 7) >> 1) + k]; };
        return as_bf16x8(__builtin_amdgcn_perm(word(eb, 0), word(ea, 0), 0x05040100u), __builtin_amdgcn_perm(word(eb, 0), word(ea, 0), 0x07060302u),
                         __builtin_amdgcn_perm(word(eb, 1), word(ea, 1), 0x05040100u), __builtin_amdgcn_perm(word(eb, 1), word(ea, 1), 0x07060302u));
    }
}

// the same from LDS: piece st of the lane's row lies at base ^ 16 st
template <int C, int KL>
__device__ __forceinline__ bf16x8_t x_in_lds(const unsigned char *lds, uint32_t base, int st)
{
    if constexpr (!PairOrder<C, KL>::value) {
        return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t *>(lds + (base ^ (uint32_t)(16 * st))));
    } else {
        const int ea = C == 4 ? 8 * st : C == 2 ? 16 * (st >> 1) + 4 * (st & 1) : 4 * st, eb = ea + 16 / C;
        const u32x2_t wa = *reinterpret_cast<const u32x2_t *>(lds + (base ^ (uint32_t)(2 * ea)));
        const u32x2_t wb = *reinterpret_cast<const u32x2_t *>(lds + (base ^ (uint32_t)(2 * eb)));
        return as_bf16x8(__builtin_amdgcn_perm(wb.x, wa.x, 0x05040100u), __builtin_amdgcn_perm(wb.x, wa.x, 0x07060302u),
                         __builtin_amdgcn_perm(wb.y, wa.y, 0x05040100u), __builtin_amdgcn_perm(wb.y, wa.y, 0x07060302u));
    }
}

template <int C, int N_COLS, bool FINE, typename X>
__device__ __forceinline__ void narrow_block(const uint32_t (&cw)[2][8], const float (&sc)[2], const float (&ze)[2],
                                             const X &x, f32x4v_t (&acc)[2])
{
    constexpr int KL = N_COLS / 4;
    const bf16x8_t ones = as_bf16x8(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    f32x4v_t d[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}}, d1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int st = 0; st < N_COLS / 32; ++st) {
        const bf16x8_t xa = x.template operand<C>(st);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            bf16x8_t b;
            if constexpr (PairOrder<C, KL>::value) b = operand_pairs<C, FINE>(cw[t], st);
            else b = operand<C, FINE>(cw[t], st);
            d[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, b, d[t], 0, 0, 0);
        }
        d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, ones, d1, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        float f = sc[t], zz = C < 8 ? fmaf(-128.0f, sc[t], ze[t]) : ze[t];
        if constexpr (FINE) term_factors<C>(sc[t], ze[t], f, zz);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = fmaf(f, d[t][r], fmaf(zz, d1[r], acc[t][r]));
    }
}

template <int KL>
struct HeldX {
    const u32x4_t (&x)[KL / 8];
    template <int C> __device__ __forceinline__ bf16x8_t operand(int st) const { return x_held<C, KL>(x, st); }
};
template <int KL>
struct StagedX {
    const unsigned char *lds;
    uint32_t base;
    template <int C> __device__ __forceinline__ bf16x8_t operand(int st) const { return x_in_lds<C, KL>(lds, base, st); }
};

template <int N_COLS, int WAVES, bool FINE, bool STAGED>
__global__ __launch_bounds__((64 * WAVES), 4)
void mp_gemm_narrow_kernel(MpArgs a)
{
    static_assert(WAVES == 8 || WAVES == 16, "sixteen partial sums");
    constexpr int SUMS = 16 / WAVES;                          // of a wave: the columns wave + WAVES s + 16 i
    constexpr int KL = N_COLS / 4, XL = KL / 8;
    constexpr int ROW = N_COLS / 8;                           // 16-byte pieces of a row of x in a block column
    constexpr int X_BYTES = STAGED ? WAVES * 16 * ROW * 16 : 0, RED_BYTES = 16 * 2 * 4 * 64 * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[X_BYTES > RED_BYTES ? X_BYTES : RED_BYTES];
    float (*const red)[2][4][64] = reinterpret_cast<float (*)[2][4][64]>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int row0 = (int)blockIdx.x * 32;                    // (R is a multiple of 32)
    const int batch0 = (int)blockIdx.y * 16, batch = a.batch - batch0;
    const int I = row0 / a.m, rin = row0 - I * a.m;
    const int64_t blk0 = a.block_base + (int64_t)I * a.nbc;
    // level and offset of this wave's t-th block column, wave + WAVES t, in lane t (512 block columns at most: 64 a wave)
    const int mine = min(wave + WAVES * lane, a.nbc - 1);
    const int lvl = a.level[blk0 + mine];
    const int64_t off = a.byte_off[blk0 + mine];
    const int nt = (a.nbc - wave + WAVES - 1) / WAVES;  // 0 or less: none
    // x: a lane's own operand (rows past the batch as the last one: not stored), or (STAGED) pieces of whole rows, by way of the
    // wave's LDS: piece c of row b at position c ^ b (64 columns: c ^ b / 2), so that 16 rows' same pieces lie in 16 different
    // quarters of the banks
    const uint16_t *const x0 = a.x + (int64_t)batch0 * a.ld_x, *const xrow = x0 + (int64_t)min(li, batch - 1) * a.ld_x + g * KL;
    const uint32_t x_at = 2u * (uint32_t)(lane / ROW) * (uint32_t)a.ld_x + 16u * (uint32_t)(lane % ROW);      // bytes
    const uint32_t x_step = 2u * (64 / ROW) * (uint32_t)a.ld_x, x_end = 2u * ((uint32_t)(min(batch, 16) - 1) * (uint32_t)a.ld_x + (uint32_t)a.C);
    unsigned char *const xl = smem + (STAGED ? wave * 16 * ROW * 16 : 0);
    const uint32_t x_to = (uint32_t)(lane * 16) ^ (uint32_t)((lane >> 4) * 16);
    const uint32_t x_from = (uint32_t)(li * ROW + ((g * XL) ^ (N_COLS == 128 ? li : li >> 1))) * 16;
    const uint32_t lane_units = (uint32_t)((rin + li) * (N_COLS / 8) + g * (KL / 8));   // x c = the lane's byte offset in the block
    const uint32_t block_bytes_per_bit = (uint32_t)a.m * (N_COLS / 8);

    struct Slot { Quarter<N_COLS> q[2]; float sc[2], ze[2]; u32x4_t x[STAGED ? 1 : XL]; int c; };
    auto request = [&](Slot &o, int t) {
        const int tt = min(t, nt - 1), J = wave + WAVES * tt;
        const int lv = __builtin_amdgcn_readlane(lvl, tt);
        int c = a.bits[0];
#pragma unroll
        for (int k = 1; k < MAX_CAND; ++k) c = lv == k ? a.bits[k] : c;
        o.c = t < nt ? c : 0;
        const uint64_t at = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)off >> 32), tt) << 32 |
                            (uint32_t)__builtin_amdgcn_readlane((uint32_t)off, tt);
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.codes) + at, 0, (int)(block_bytes_per_bit * (uint32_t)o.c), 0x00027000);
        const float *ps = a.scale + (blk0 + J) * a.m + rin, *pz = a.zero + (blk0 + J) * a.m + rin;
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) load_quarter<N_COLS>(rs, (lane_units + (uint32_t)(tl * 16 * (N_COLS / 8))) * (uint32_t)o.c, o.q[tl]);
        if constexpr (!STAGED) {
#pragma unroll
            for (int i = 0; i < XL; ++i) o.x[i] = *(const __attribute__((address_space(1))) u32x4_t *)(xrow + J * N_COLS + 8 * i);
        }
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
            o.sc[tl] = ps[16 * tl + li];
            o.ze[tl] = pz[16 * tl + li];
        }
    };
    // STAGED: x of one block at a time on the way (it comes from the caches); what lies past the rows reads as zero
    u32x4_t xr[STAGED ? XL : 1];
    auto request_x = [&](int t) {
        if constexpr (STAGED) {
            const int J = wave + WAVES * min(t, nt - 1);
            const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x0 + J * N_COLS), 0, (int)(x_end - 2u * (uint32_t)(J * N_COLS)), 0x00027000);
#pragma unroll
            for (int i = 0; i < XL; ++i) xr[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(x_at + (uint32_t)i * x_step), 0, 0));
        }
    };
    auto stage_x = [&]() {
        if constexpr (STAGED) {
            // (a wave's LDS accesses are done in order: the fences keep the compiler to it)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint32_t to = x_to;                               // (addresses made here, not kept for all blocks)
            asm volatile("" : "+v"(to));
#pragma unroll
            for (int i = 0; i < XL; ++i) *reinterpret_cast<u32x4_t *>(xl + (to ^ (uint32_t)(i * (1024 + 64)))) = xr[i];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    f32x4v_t sums[SUMS][2];
#pragma unroll
    for (int s = 0; s < SUMS; ++s)
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) sums[s][tl] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};
    auto add = [&](const Slot &o, f32x4v_t (&acc)[2]) {
        if (o.c == 0) return;                                 // no such block column, or a pruned block
        uint32_t cw[2][8];
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
            uint32_t r[N_COLS / 16];
            align_quarter<N_COLS>(o.q[tl], (lane_units + (uint32_t)(tl * 16 * (N_COLS / 8))) * (uint32_t)o.c, r);
#pragma unroll
            for (int i = 0; i < N_COLS / 16; ++i) cw[tl][i] = r[i];
        }
        if constexpr (STAGED) {
            uint32_t from = x_from;                           // (addresses made here, not kept for all blocks)
            asm volatile("" : "+v"(from));
            const StagedX<KL> x{xl, from};
#define ND_BLOCK(C) narrow_block<C, N_COLS, FINE>(cw, o.sc, o.ze, x, acc)
            MP_SWITCH(o.c, ND_BLOCK)
        } else {
            const HeldX<KL> x{o.x};
            MP_SWITCH(o.c, ND_BLOCK)
#undef ND_BLOCK
        }
    };
    if (nt > 0) {
        Slot s0, s1;
        request(s0, 0);
        request_x(0);
        request(s1, 1);
        for (int t = 0; t < nt; t += 2) {
            stage_x();
            request_x(t + 1);
            add(s0, sums[0]);
            if (t + 2 < nt) request(s0, t + 2);
            stage_x();
            if (t + 2 < nt) request_x(t + 2);
            add(s1, sums[SUMS - 1]);
            if (t + 2 < nt) request(s1, t + 3);
        }
    }
    if constexpr (STAGED) __syncthreads();                    // every wave is done with its x
#pragma unroll
    for (int s = 0; s < SUMS; ++s)
#pragma unroll
        for (int tl = 0; tl < 2; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave + WAVES * s][tl][r][lane] = sums[s][tl][r];
    __syncthreads();
    // D layout: batch row 4 (lane / 16) + r, channel lane % 16
    const int ch = tid & 31, b = tid >> 5;                    // 32 channels x 16 batch rows in the first 512 threads
    if (b < batch && b < 16) {
        float v = red[0][ch >> 4][b & 3][(b >> 2) * 16 + (ch & 15)];
#pragma unroll
        for (int w = 1; w < 16; ++w) v = v + red[w][ch >> 4][b & 3][(b >> 2) * 16 + (ch & 15)];
        a.out[(int64_t)(batch0 + b) * a.R + row0 + ch] = v;
    }
}

// ================================================================ more than 32 batch rows
// A workgroup takes CT tiles of 16 channels and NB tiles of 16 batch rows; its WAVES waves take every WAVES-th block column each and
// share nothing but the sum at the end, so no barrier holds them in step.  A wave brings the x of its next block column into LDS of
// its own by direct loads (whole rows, 1 KiB a load), reads all operands of the present one into registers (64 of them, at 4 batch tiles and
// 128 columns) and then asks for the next: x is read from LDS once per wave.
// Codes of a pair of tiles are asked for a block ahead, into the registers that the pair has just done with.  Bitwidths and
// offsets lie in LDS from the start.  sum_j x of the block comes from a product with ones, per wave (16 of its 80 matrix
// instructions at 4 x 4 tiles).
// Vector issue bounds it: at 4 x 4 tiles and 128 columns unpacking 64 codes in pairs takes 128 .. 192 instructions a lane and block,
// two FMAs per output 128; next are the direct loads of x, which take a wave 40 clocks each to ask for (8192 x 28672 at 128 rows
// without them 88 us instead of 102).  Tiles of 64 x 64 are the largest whose sums, operands and codes fit 256
// registers.  With 8 waves a workgroup has the CU to itself; with 4, two of them take turns in starting and ending.
// Its predecessor held 8 waves in step, a barrier a step, x read from LDS once per 32 channels.  Against that one: 14336 x 4096 at 100
// rows, bitwidths 1 .. 8, 39.0 -> 30.6 us; 8192 x 28672 at 128 rows 139 -> 92; 14336 x 4096 in 64-column blocks at 100 rows 55.7 -> 39.2;
// 4096 x 4096 at 64 rows 12.9 -> 10.1; in 41 drawn products of which the estimates had said the contrary it takes 0.88 of the time, 0.95 at most.

// one tile of 16 channels and NB tiles of 16 batch rows: the block's products, scale and zero applied
template <int C, int N_COLS, int NB>
__device__ __forceinline__ void many_tile(const uint32_t (&cw)[N_COLS / 16], float sc, float ze, const u32x4_t (&x)[NB][N_COLS / 32],
                                          const f32x4v_t (&s)[NB], f32x4v_t (&acc)[NB])
{
    constexpr int STEPS = N_COLS / 32;
    const f32x4v_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4v_t d[NB];
    uint32_t one = PairConst<C>::one, mask = PairConst<C>::field | PairConst<C>::field << 16;
    asm volatile("" : "+v"(one), "+s"(mask));
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        uint32_t o[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) o[p] = code_pair<C>(cw, 8 * st + 2 * p, one, mask);
        const bf16x8_t b = as_bf16x8(o[0], o[1], o[2], o[3]);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            d[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[nb][st]), b, st == 0 ? zero4 : d[nb], 0, 0, 0);
    }
    float f, z;
    term_factors<C>(sc, ze, f, z);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[nb][r] = fmaf(f, d[nb][r], fmaf(z, s[nb][r], acc[nb][r]));
}

// Two tiles at 1 bit, unless ONE_BIT_FINE (an instance of its own: a choice in the kernel cost the other widths 3 .. 5 %): 128 + q and columns in the order of the kernel for up to 32 rows (pair order for 128 columns), with sums of x of
// their own.  What a row of x gives then differs little between that kernel and this one (14336 x 4096, bitwidths 1 .. 8: by 1.3e-4 of the root
// mean square at most, 4.3e-4 with 1 + q / 2 here), but both are 1e-5 from the exact product, by the norm, where 1 + q / 2 would be 3e-7: see
// one_bit_line.
template <int N_COLS, int NB>
__device__ __forceinline__ void many_tiles_1bit(const uint32_t (&cw)[2][N_COLS / 16], const float *sc, const float *ze,
                                                const u32x4_t (&x)[NB][N_COLS / 32], f32x4v_t (&acc0)[NB], f32x4v_t (&acc1)[NB])
{
    constexpr int STEPS = N_COLS / 32, KL = N_COLS / 4;
    const f32x4v_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    const bf16x8_t ones = as_bf16x8(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    bf16x8_t b[2][STEPS];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            uint32_t o[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if constexpr (N_COLS == 128) o[p] = ((cw[t][0] >> (4 * st + p)) & 0x00010001u) | 0x43004300u;
                else o[p] = ((cw[t][0] >> (8 * st + 2 * p)) & 1u) | ((cw[t][0] >> (8 * st + 2 * p + 1)) & 1u) << 16 | 0x43004300u;
            }
            b[t][st] = as_bf16x8(o[0], o[1], o[2], o[3]);
        }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        f32x4v_t d0 = zero4, d1 = zero4, s1 = zero4;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const bf16x8_t xa = x_held<1, KL>(x[nb], st);
            d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, b[0][st], d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, b[1][st], d1, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, ones, s1, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            acc0[nb][r] = fmaf(sc[0], fmaf(-128.0f, s1[r], d0[r]), fmaf(ze[0], s1[r], acc0[nb][r]));
            acc1[nb][r] = fmaf(sc[1], fmaf(-128.0f, s1[r], d1[r]), fmaf(ze[1], s1[r], acc1[nb][r]));
        }
        __builtin_amdgcn_sched_barrier(0);                    // (registers: a batch tile at a time)
    }
}

// all operands of a block of 128 (STEPS = 4) or 64 columns, NB batch tiles, at: the lane's first one; and 16 bytes at meta_at
template <int NB, int STEPS>
__device__ __forceinline__ void read_block(uint32_t at, uint32_t meta_at, u32x4_t (&x)[NB][STEPS], u32x4_t &meta)
{
    static_assert(NB >= 2 && NB <= 4 && (STEPS == 2 || STEPS == 4), "written out");
    if constexpr (STEPS == 4 && NB == 4)
        asm volatile("ds_read_b128 %0, %18\n\tds_read_b128 %1, %17\n\tds_read_b128 %2, %17 offset:16\n\t"
                     "ds_read_b128 %3, %17 offset:32\n\tds_read_b128 %4, %17 offset:48\n\tds_read_b128 %5, %17 offset:4160\n\t"
                     "ds_read_b128 %6, %17 offset:4176\n\tds_read_b128 %7, %17 offset:4192\n\tds_read_b128 %8, %17 offset:4208\n\t"
                     "ds_read_b128 %9, %17 offset:8320\n\tds_read_b128 %10, %17 offset:8336\n\tds_read_b128 %11, %17 offset:8352\n\t"
                     "ds_read_b128 %12, %17 offset:8368\n\tds_read_b128 %13, %17 offset:12480\n\t"
                     "ds_read_b128 %14, %17 offset:12496\n\tds_read_b128 %15, %17 offset:12512\n\t"
                     "ds_read_b128 %16, %17 offset:12528\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[1][0]), 
                       "=&v"(x[1][1]), "=&v"(x[1][2]), "=&v"(x[1][3]), "=&v"(x[2][0]), "=&v"(x[2][1]), "=&v"(x[2][2]), 
                       "=&v"(x[2][3]), "=&v"(x[3][0]), "=&v"(x[3][1]), "=&v"(x[3][2]), "=&v"(x[3][3])
                     : "v"(at), "v"(meta_at) : "memory");
    else if constexpr (STEPS == 4 && NB == 3)
        asm volatile("ds_read_b128 %0, %14\n\tds_read_b128 %1, %13\n\tds_read_b128 %2, %13 offset:16\n\t"
                     "ds_read_b128 %3, %13 offset:32\n\tds_read_b128 %4, %13 offset:48\n\tds_read_b128 %5, %13 offset:4160\n\t"
                     "ds_read_b128 %6, %13 offset:4176\n\tds_read_b128 %7, %13 offset:4192\n\tds_read_b128 %8, %13 offset:4208\n\t"
                     "ds_read_b128 %9, %13 offset:8320\n\tds_read_b128 %10, %13 offset:8336\n\tds_read_b128 %11, %13 offset:8352\n\t"
                     "ds_read_b128 %12, %13 offset:8368\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[1][0]), 
                       "=&v"(x[1][1]), "=&v"(x[1][2]), "=&v"(x[1][3]), "=&v"(x[2][0]), "=&v"(x[2][1]), "=&v"(x[2][2]), 
                       "=&v"(x[2][3])
                     : "v"(at), "v"(meta_at) : "memory");
    else if constexpr (STEPS == 4 && NB == 2)
        asm volatile("ds_read_b128 %0, %10\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %9 offset:16\n\t"
                     "ds_read_b128 %3, %9 offset:32\n\tds_read_b128 %4, %9 offset:48\n\tds_read_b128 %5, %9 offset:4160\n\t"
                     "ds_read_b128 %6, %9 offset:4176\n\tds_read_b128 %7, %9 offset:4192\n\tds_read_b128 %8, %9 offset:4208\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[1][0]), 
                       "=&v"(x[1][1]), "=&v"(x[1][2]), "=&v"(x[1][3])
                     : "v"(at), "v"(meta_at) : "memory");
    else if constexpr (STEPS == 2 && NB == 4)
        asm volatile("ds_read_b128 %0, %10\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %9 offset:16\n\t"
                     "ds_read_b128 %3, %9 offset:2080\n\tds_read_b128 %4, %9 offset:2096\n\tds_read_b128 %5, %9 offset:4160\n\t"
                     "ds_read_b128 %6, %9 offset:4176\n\tds_read_b128 %7, %9 offset:6240\n\tds_read_b128 %8, %9 offset:6256\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), 
                       "=&v"(x[2][1]), "=&v"(x[3][0]), "=&v"(x[3][1])
                     : "v"(at), "v"(meta_at) : "memory");
    else if constexpr (STEPS == 2 && NB == 3)
        asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %7\n\tds_read_b128 %2, %7 offset:16\n\t"
                     "ds_read_b128 %3, %7 offset:2080\n\tds_read_b128 %4, %7 offset:2096\n\tds_read_b128 %5, %7 offset:4160\n\t"
                     "ds_read_b128 %6, %7 offset:4176\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), 
                       "=&v"(x[2][1])
                     : "v"(at), "v"(meta_at) : "memory");
    else if constexpr (STEPS == 2 && NB == 2)
        asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %5 offset:16\n\t"
                     "ds_read_b128 %3, %5 offset:2080\n\tds_read_b128 %4, %5 offset:2096\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(meta), "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1])
                     : "v"(at), "v"(meta_at) : "memory");
}

template <int N_COLS, int NB, int CT, int WAVES, bool ONE_BIT_FINE>
__global__ __launch_bounds__((64 * WAVES), 2)
void mp_gemm_many_kernel(MpArgs a, int cols_per_split)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    constexpr int KL = N_COLS / 4, STEPS = N_COLS / 32;
    constexpr int CHUNKS = N_COLS / 8, RPL = 64 / CHUNKS;     // 16-byte chunks of a row; rows of a load
    constexpr int ROWS = NB * 16, LOADS = ROWS / RPL, XB = LOADS * 1040;     // batch rows; loads and bytes of x of a wave
    constexpr int H = CT / 2, ENTRIES = 32768 / N_COLS / WAVES;         // (of a wave)
    static_assert(CT % 2 == 0, "pairs of tiles");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int batch0 = (int)blockIdx.z * ROWS, batch = min(a.batch - batch0, ROWS);
    const int row0 = (int)blockIdx.x * (CT * 16);
    const int J0 = (int)blockIdx.y * cols_per_split, J1 = min(J0 + cols_per_split, a.nbc);
    const int nt = (J1 - J0 - wave + WAVES - 1) / WAVES;                     // this wave's block columns: 0 or less: none
    const int turn0 = nt > 1 ? (int)(blockIdx.x >> 3) & 1 : 0;    // (rows of x may lie a power of two apart: not all at the same columns)
    auto nth = [&](int t) { const int u = turn0 + t; return u < nt ? u : u - nt; };

    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t lds0 = lds_base + (uint32_t)(wave * XB), meta0 = lds_base + (uint32_t)(WAVES * XB + wave * (ENTRIES * 16));
    // the lane, as new each time: what follows from it is made again where it is needed, not kept in registers
    auto fresh_lane = [&]() { uint32_t l = (uint32_t)lane; asm volatile("" : "+v"(l)); return l; };

    // this wave's blocks: offsets, and bitwidths (0: past the matrix, or pruned) in their upper bytes, in LDS: 16 bytes a block column
    int rin[H];
    const float *scale0[H], *zero0[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int r = row0 + 32 * h;
        const bool ok = r < a.R;
        const int I = ok ? r / a.m : 0;
        rin[h] = ok ? r - I * a.m : 0;
        const int64_t blk0 = a.block_base + (int64_t)I * a.nbc;
        scale0[h] = a.scale + blk0 * a.m + rin[h];
        zero0[h] = a.zero + blk0 * a.m + rin[h];
        for (int e = lane; e < nt; e += 64) {                 // (nt <= ENTRIES: a matrix has 32768 columns at most)
            const int64_t b = blk0 + J0 + wave + WAVES * e;
            const int lv = a.level[b];
            const int64_t off = a.byte_off[b];
            int c = a.bits[0];
#pragma unroll
            for (int k = 1; k < MAX_CAND; ++k) c = lv == k ? a.bits[k] : c;
            *reinterpret_cast<uint64_t *>(smem + WAVES * XB + (wave * ENTRIES + e) * 16 + h * 8) = (uint64_t)off | (uint64_t)(uint32_t)(ok ? c : 0) << 56;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    auto meta_at = [&](int t) { return meta0 + (uint32_t)nth(min(t, nt - 1)) * 16; };

    // x: a load's rows at positions that differ, the next load's 16 bytes further: 16 rows' same chunk in 16 different quarters of the banks
    const uint32_t ldx2 = 2u * (uint32_t)a.ld_x;
    const rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x) + (int64_t)batch0 * a.ld_x, 0,
                                                         (int)((uint32_t)(batch - 1) * ldx2 + 2u * (uint32_t)a.C), 0x00027000);
    auto fetch = [&](int t) {
        const int J = J0 + wave + WAVES * nth(min(t, nt - 1));
        const uint32_t l = fresh_lane(), lrow = l / CHUNKS, lpos = l % CHUNKS;
        const uint32_t vrow = __umul24(lrow, ldx2) + (lpos ^ (N_COLS == 128 ? lrow * 4 : (lrow >> 1) * 2)) * 16u;
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (__attribute__((address_space(3))) void *)(lds0 + (uint32_t)(i * 1040)),
                                                     16, (int)(vrow + (uint32_t)(i * RPL) * ldx2), J * N_COLS * 2, 0, 0);
    };
    auto x_at = [&]() {
        const uint32_t l = fresh_lane(), i = l & 15, q = l >> 4;
        return lds0 + (N_COLS == 128 ? (i >> 2) * 1040 + (i & 3) * 256 + (q ^ (i & 3)) * 64
                                     : (i >> 3) * 1040 + (i & 7) * 128 + (q ^ ((i >> 1) & 3)) * 32);
    };

    Quarter<N_COLS> cq[CT];
    float sc[CT], ze[CT];
    int cb[H];
    const uint32_t block_bytes_per_bit = (uint32_t)a.m * (N_COLS / 8);
    // x c = the lane's byte offset in the block
    const uint32_t units0 = (uint32_t)(li * (N_COLS / 8) + g * (KL / 8));
    auto units = [&](int h) {
        return units0 + (uint32_t)(rin[h] * (N_COLS / 8));
    };
    auto request = [&](int h, int t, uint32_t hi, uint32_t lo) {
        const int J = J0 + wave + WAVES * nth(min(t, nt - 1));
        const uint32_t c = t < nt ? hi >> 24 : 0;
        cb[h] = (int)c;
        const uint64_t at = (uint64_t)(hi & 0xffffffu) << 32 | lo;
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.codes) + at, 0, (int)(block_bytes_per_bit * c), 0x00027000);
        const float *ps = scale0[h] + (uint32_t)(J * a.m), *pz = zero0[h] + (uint32_t)(J * a.m);
        const uint32_t u = units(h), i = (uint32_t)li;
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) load_quarter<N_COLS>(rs, __umul24(u + (uint32_t)(tl * 16 * (N_COLS / 8)), c), cq[2 * h + tl]);
        sc[2 * h] = ps[i]; sc[2 * h + 1] = (ps + 16)[i];
        ze[2 * h] = pz[i]; ze[2 * h + 1] = (pz + 16)[i];
    };

    const f32x4v_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    const bf16x8_t ones = as_bf16x8(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
    f32x4v_t acc[CT][NB];
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[t][nb] = zero4;
    if (nt > 0) {
        fetch(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        u32x4_t meta;
        uint32_t mw[4];
        auto scalars = [&]() {
            mw[0] = (uint32_t)__builtin_amdgcn_readfirstlane(meta.x); mw[1] = (uint32_t)__builtin_amdgcn_readfirstlane(meta.y);
            mw[2] = (uint32_t)__builtin_amdgcn_readfirstlane(meta.z); mw[3] = (uint32_t)__builtin_amdgcn_readfirstlane(meta.w);
        };
        asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(meta) : "v"(meta_at(0)) : "memory");
        scalars();
#pragma unroll
        for (int h = 0; h < H; ++h) request(h, 0, mw[2 * h + 1], mw[2 * h]);
        for (int t = 0; t < nt; ++t) {
            u32x4_t x[NB][STEPS];
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(8 * H) : "memory");     // x is there: the codes requested behind it may be on their way
            read_block<NB, STEPS>(x_at(), meta_at(t + 1), x, meta);    // (read: its place is free)
            scalars();
            __builtin_amdgcn_sched_barrier(0);
            fetch(t + 1);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            f32x4v_t s[NB];
#pragma unroll
            for (int st = 0; st < STEPS; ++st)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    s[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[nb][st]), ones, st == 0 ? zero4 : s[nb], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                uint32_t cw[2][N_COLS / 16];
#pragma unroll
                for (int tl = 0; tl < 2; ++tl)
                    align_quarter<N_COLS>(cq[2 * h + tl], N_COLS == 128 ? 0 : __umul24(units(h) + (uint32_t)(tl * 16 * (N_COLS / 8)), (uint32_t)cb[h]), cw[tl]);
#define MB_TILE(C)                                                                                                \
    do {                                                                                                          \
        if constexpr (C == 1 && !ONE_BIT_FINE) {                                                                  \
            many_tiles_1bit<N_COLS, NB>(cw, sc + 2 * h, ze + 2 * h, x, acc[2 * h], acc[2 * h + 1]);               \
        } else {                                                                                                  \
            many_tile<C, N_COLS, NB>(cw[0], sc[2 * h], ze[2 * h], x, s, acc[2 * h]);                              \
            many_tile<C, N_COLS, NB>(cw[1], sc[2 * h + 1], ze[2 * h + 1], x, s, acc[2 * h + 1]);                  \
        }                                                                                                         \
    } while (0)
                MP_SWITCH(cb[h], MB_TILE)
#undef MB_TILE
                request(h, t + 1, mw[2 * h + 1], mw[2 * h]);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                          // every wave is done with its x
    // the waves add up, in a fixed order
    float *red = reinterpret_cast<float *>(smem);             // [wave][tile][nb][lane][4]
#pragma unroll
    for (int tl = 0; tl < CT; ++tl)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            *reinterpret_cast<f32x4v_t *>(red + (((wave * CT + tl) * NB + nb) * 64 + lane) * 4) = acc[tl][nb];
    __syncthreads();
    float *dst = a.out + ((int64_t)blockIdx.y * a.batch + batch0) * a.R;
    for (int p = wave; p < CT * NB; p += WAVES) {
        const int tl = p / NB, nb = p % NB;
        if (row0 + 16 * tl >= a.R) continue;
        f32x4v_t v = *reinterpret_cast<const f32x4v_t *>(red + (p * 64 + lane) * 4);
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v = v + *reinterpret_cast<const f32x4v_t *>(red + ((w * CT * NB + p) * 64 + lane) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int b = 16 * nb + 4 * g + r;
            if (b < batch) dst[(int64_t)b * a.R + row0 + 16 * tl + li] = v[r];
        }
    }
}

// y = sum over the column splits of the partials, split 0 first
__global__ __launch_bounds__(256)
void mp_gemm_finish_kernel(const float *__restrict__ part, int64_t n, int n_split, float *__restrict__ y)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float v = part[i];
    for (int s = 1; s < n_split; ++s) v = v + part[(int64_t)s * n + i];
    y[i] = v;
}

}  // namespace sbits

using namespace sbits;

int sbits_mp_gemm_splits(int64_t cols, int n) { return (int)((cols / n + MG_SPAN - 1) / MG_SPAN); }

bool sbits_mp_gemm_shapes_ok(const sbits_plan *plan)
{
    return (plan->n == 64 || plan->n == 128) && plan->m % 32 == 0;
}

// Shapes of the kernel of many rows, and what a product takes in each, in microseconds: fitted to 1350
// products of 256 .. 28672 rows and columns, 33 .. 128 rows of x, in all shapes and column splits (mean error 3 .. 7 %; the shape
// chosen by them is 2 % behind the best one on average).  turns: of workgroups on 256 CUs, one a CU or, with four
// waves, two; work: block columns of a wave times workgroups of a CU.  The choice decides the order of the sums, so it goes by the matrix
// and the batch, for a whole device.  Less than 6 us, little more than a launch, is not promised.
struct ManyShape { int nb, ct, waves; double base, turn, col, col_bit, split, per_split, part, turn_col; };
static const ManyShape MANY_128[5] = {{2, 2, 8, 4.263, 0.231, 0.853, 0.029, 2.233, 0.113, 0.0, 0.0},
                                      {3, 2, 8, 2.786, 1.491, 1.304, 0.013, 1.997, 0.157, 0.736, 0.0},
                                      {3, 4, 4, 2.899, 1.947, 0.889, 0.0, 1.449, 0.220, 1.920, 0.541},
                                      {4, 4, 4, 2.875, 2.236, 1.168, 0.0, 1.379, 0.239, 2.000, 0.551},
                                      {4, 4, 8, 1.635, 2.728, 2.833, 0.0, 1.534, 0.240, 1.923, 0.0}};
static const ManyShape MANY_64[5] = {{2, 2, 8, 3.597, 0.950, 0.536, 0.030, 2.402, 0.120, 0.0, 0.0},
                                     {3, 2, 8, 4.009, 0.430, 0.719, 0.025, 2.285, 0.133, 0.0, 0.0},
                                     {3, 4, 4, 4.873, 0.0, 0.490, 0.0, 1.520, 0.197, 1.805, 0.545},
                                     {4, 4, 4, 3.332, 1.874, 0.636, 0.0, 1.306, 0.206, 2.053, 0.572},
                                     {4, 4, 8, 1.973, 2.905, 1.799, 0.0, 1.303, 0.213, 1.870, 0.0}};
static ManySplit many_split(const sbits_plan *plan, int64_t R, int nbc, int tiles)     // (all that counts of the batch: the workspace is sized by them)
{
    const ManyShape *const shapes = plan->n == 128 ? MANY_128 : MANY_64;
    double bits = 0;
    for (int l = 0; l < plan->K; ++l) bits += plan->bits[l];
    bits /= plan->K;
    ManySplit best = {0, nbc, 1, 1e30};
    for (int f = 0; f < 5; ++f) {
        const ManyShape &s = shapes[f];
        if (s.nb > tiles) continue;
        const int64_t wgs1 = (R + s.ct * 16 - 1) / (s.ct * 16) * ((tiles + s.nb - 1) / s.nb);
        for (int sp : {1, 2, 3, 4, 6, 8, 12, 16}) {
            if (sp > 1 && (wgs1 * sp > 600 || nbc < 2 * sp)) break;
            const int per = (nbc + sp - 1) / sp, n_split = (nbc + per - 1) / per;
            const int64_t wgs = wgs1 * n_split, of_cu = (wgs + 255) / 256, at_once = s.waves == 4 ? 2 : 1;
            const double turns = (double)((of_cu + at_once - 1) / at_once), cols = (per + s.waves - 1) / s.waves;
            double us = s.base + turns * (s.turn + s.turn_col * cols) + (double)of_cu * cols * (s.col + s.col_bit * bits);
            if (n_split > 1) us += s.split + s.per_split * n_split + s.part * 1e-6 * (double)(tiles * 16 * R * n_split);
            if (us < 6.0) us = 6.0;
            if (us < best.us) best = {f, per, n_split, us};
        }
    }
    return best;
}

// the choice for 33 .. 128 rows of each matrix, made with the plan: 40 estimates are too many for a call of a few microseconds
void sbits_mp_gemm_tables(sbits_plan *plan)
{
    if (!sbits_mp_gemm_shapes_ok(plan)) return;
    for (int i = 0; i < plan->n_mats; ++i) {
        int same = 0;
        while (same < i && same < 16 && (plan->rows[same] != plan->rows[i] || plan->cols[same] != plan->cols[i])) ++same;
        for (int tiles = 3; tiles <= 8; ++tiles)
            plan->many.push_back(same < i && same < 16 ? plan->many[(size_t)same * 6 + tiles - 3]
                                                       : many_split(plan, plan->rows[i], (int)(plan->cols[i] / plan->n), tiles));
    }
}
static const ManySplit &many_of(const sbits_plan *plan, int mat, int batch) { return plan->many[(size_t)mat * 6 + (size_t)((batch + 15) / 16 - 3)]; }

// partial sums of the largest matrix: 32 rows of the first kernel, and each number of tiles of the one for many rows
size_t sbits_mp_gemm_ws_bytes(const sbits_plan *plan)
{
    if (!sbits_mp_gemm_shapes_ok(plan)) return 0;
    size_t mx = 0;
    for (int i = 0; i < plan->n_mats; ++i) {
        auto need = [&](int splits, int batch) {
            const size_t b = splits > 1 ? (size_t)splits * batch * (size_t)plan->rows[i] * 4 : 0;
            if (b > mx) mx = b;
        };
        need(sbits_mp_gemm_splits(plan->cols[i], plan->n), 32);
        for (int tiles = 3; tiles <= 8; ++tiles) need(many_of(plan, i, tiles * 16).n_split, tiles * 16);
    }
    return sbits_align_up(mx, 256);
}

template <int N_COLS, int NB, int RG, bool FINE>
static int launch_mp(sbits_ctx *ctx, const MpArgs &a)
{
    constexpr size_t x_bytes = (size_t)16 * NB * (MG_SPAN * N_COLS * 2 + 16);
    constexpr size_t red_bytes = (size_t)MG_JL * RG * 2 * NB * 4 * 64 * 4;
    constexpr size_t lds = x_bytes > red_bytes ? x_bytes : red_bytes;
    auto *fn = &mp_gemm_kernel<N_COLS, NB, RG, FINE>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds));
    const dim3 grid((unsigned)((a.R + RG * 32 - 1) / (RG * 32)), (unsigned)a.n_split);
    hipLaunchKernelGGL(fn, grid, dim3(64 * MG_JL * RG), lds, ctx->stream, a);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

template <int N_COLS, int WAVES, bool FINE, bool STAGED>
static int launch_narrow(sbits_ctx *ctx, const MpArgs &a)
{
    const dim3 grid((unsigned)(a.R / 32), (unsigned)((a.batch + 15) / 16));
    hipLaunchKernelGGL((mp_gemm_narrow_kernel<N_COLS, WAVES, FINE, STAGED>), grid, dim3(64 * WAVES), 0, ctx->stream, a);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

template <int N_COLS, int NB, int CT, int WAVES, bool FINE>
static int launch_many(sbits_ctx *ctx, const MpArgs &a, const ManySplit &ms)
{
    constexpr size_t x = (size_t)WAVES * NB * 16 * N_COLS * 2 / 1024 * 1040, red = (size_t)WAVES * CT * NB * 1024;
    constexpr size_t all = x + (size_t)(32768 / N_COLS) * 16, lds = all > red ? all : red;      // (and the waves' tables of their blocks)
    auto *fn = &mp_gemm_many_kernel<N_COLS, NB, CT, WAVES, FINE>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const dim3 grid((unsigned)((a.R + CT * 16 - 1) / (CT * 16)), (unsigned)ms.n_split, (unsigned)((a.batch + NB * 16 - 1) / (NB * 16)));
    hipLaunchKernelGGL(fn, grid, dim3(64 * WAVES), lds, ctx->stream, a, ms.per_split);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

template <int N_COLS, bool FINE>
static int launch_many_shape(sbits_ctx *ctx, const MpArgs &a, const ManySplit &ms)      // (the order of MANY_128 and MANY_64)
{
    switch (ms.shape) {
    case 0: return launch_many<N_COLS, 2, 2, 8, FINE>(ctx, a, ms);
    case 1: return launch_many<N_COLS, 3, 2, 8, FINE>(ctx, a, ms);
    case 2: return launch_many<N_COLS, 3, 4, 4, FINE>(ctx, a, ms);
    case 3: return launch_many<N_COLS, 4, 4, 4, FINE>(ctx, a, ms);
    default: return launch_many<N_COLS, 4, 4, 8, FINE>(ctx, a, ms);
    }
}

// What a product takes in the first kernel (up to 32 rows) and in the narrow one (up to 64), in microseconds, fitted to 2600 and
// 900 products of 256 .. 28672 x 256 .. 28672, 1 .. 64 rows of x, bitwidths up to 8.  With the choice made by these, 1400 others of
// the same ranges took 1.3 .. 1.5 % longer on average than with the better kernel each time, 23 % at most (always the first, or
// above 32 rows this one's predecessor for many, 14 %; always the narrow one 10 .. 12 %); no product takes less than a launch, 5.2.  (The turns are
// those of a whole device also on a partition of one, here and in one_bit_line: the choice decides the order of the sums, and a
// product gives the same bits on either.)
// First: by the turns of the CUs (32 channels and 16 block columns each, 256 at a time) and their bytes; with several column
// splits, their number, the partial sums and the second launch (1024 x 17216 in 64-column blocks, 17 splits, 12.5 us).
// Narrow: by turns of 256 workgroups and block columns in each, x once more per turn; with 17 rows or more a workgroup per
// 16 of them (4096 x 4096 at 32 rows: 11.5 us in the first kernel and 6.9 in this one; 14336 x 4096 15.5 and 17.8).
struct FewRows { double first, narrow; };
static FewRows few_rows(const sbits_plan *plan, int64_t R, int nbc, int batch)
{
    const bool wide = plan->n == 128;
    const int groups = (batch + 15) / 16, b = batch < 16 ? batch : 16, splits = (nbc + MG_SPAN - 1) / MG_SPAN;
    const double turns = (double)((R / 32 * groups + 255) / 256 - 1);         // beyond the first
    const double load = (double)(R / 32 * splits) / 256, over = load > 1 ? load - 1 : 0;
    double bits = 0;                                          // of the candidates, on average
    for (int l = 0; l < plan->K; ++l) bits += plan->bits[l];
    bits /= plan->K;
    FewRows o;
    if (splits == 1) {
        if (wide) {
            o.narrow = 5.27 + 0.0325 * nbc + turns * (0.364 + nbc * (0.0065 * b + 0.0105 * bits - 0.0152));
            o.first = batch <= 16 ? 5.62 + 0.032 * nbc + over * (0.28 + nbc * (0.048 + 0.020 * bits))
                                  : 6.45 + 0.15 * nbc + over * (0.67 + nbc * (0.044 * bits - 0.071));
        } else {
            o.narrow = 5.53 + 0.0064 * nbc + turns * (0.353 + nbc * (0.0044 * b + 0.0034 * bits - 0.0085));
            o.first = batch <= 16 ? 5.68 + 0.003 * nbc + over * (nbc * (0.045 + 0.0079 * bits) - 0.23)
                                  : 5.45 + 0.058 * nbc + over * (0.55 + nbc * (0.055 + 0.0087 * bits));
        }
    } else {
        const double part = (double)batch * (double)R * splits * 1e-6;        // partial sums, millions
        if (wide) {
            o.narrow = 3.34 + 0.0333 * b + nbc * (0.101 + 0.0006 * b) + turns * (0.73 + nbc * (0.0503 + 0.0011 * b + 0.011 * bits));
            o.first = batch <= 16 ? 7.75 + 0.236 * splits + 1.98 * over + load * (0.155 * bits - 0.77) + 3.79 * part
                                  : 10.6 + 0.249 * splits + 2.75 * over + load * (0.244 * bits - 1.26) + 1.89 * part;
            // at a draw the first: where its workgroups (128 channels, alone on a CU) fill whole turns it is faster than fitted, 8192 x 8192
            // at 32 rows 16.6 .. 18.1 us and 18.5 .. 20.6 in the narrow one.  Where they just miss one it is slower (6912 x 10496 at 31 rows
            // 27.7 and 22.5).  Over 604 drawn products of this kind the choice is 0.85 % behind the better kernel with the margin and
            // 0.72 % without: it stands for the shapes that fill their turns.
            if (batch > 16 && turns > 0) o.narrow *= 1.12;
        } else {
            o.narrow = 3.32 + 0.033 * b + nbc * 0.0775 + turns * (0.40 + nbc * (0.0448 + 0.0005 * b + 0.0101 * bits));
            o.first = batch <= 16 ? 7.51 + 0.217 * splits + 1.90 * over + load * (0.082 * bits - 0.91) + 2.01 * part
                                  : 7.69 + 0.254 * splits + 1.61 * over + load * (0.072 * bits - 0.43) + 2.15 * part;
        }
    }
    if (o.first < 5.2) o.first = 5.2;
    if (o.narrow < 5.2) o.narrow = 5.2;
    return o;
}

// Up to 16 block columns and two turns of the narrow kernel, where both take hardly more than a launch, it is the better one (up to
// 16 rows by 3 .. 8 % on average and at most 3 % slower, up to 32 by 5 .. 26 %).
// Above 32 rows: against the kernel of many rows, where codes of 1 bit have the offset that they have here on this side of one_bit_line (6368 x 2624
// at 33 rows, 1 .. 4 bits, 15.3 us here and 8.9 there: the line alone had them here); on the other side that kernel takes them all.
// A pitch of x past the 32-bit offsets of the narrow kernel: the first.
static bool has_one_bit(const sbits_plan *plan)
{
    for (int l = 0; l < plan->K; ++l)
        if (plan->bits[l] == 1) return true;
    return false;
}

// Where codes of 1 bit enter as 1 + q / 2 and where as 128 + q is part of what a product of 33 .. 96 rows gives: by the norm it is 3e-7 from the
// exact one, or 1e-5; in single values the two differ by up to 3e-4 of the root mean square, with outlier channels by up to 4e-3.  So this line
// stays where it was drawn, when 128 + q was all that the kernel of many rows had: by the time, in hundredths of a microsecond above the launch, that
// a product took in that kernel's predecessor: 8 waves, 128 or 64 channels and 4 or 2 block columns a step, two steps at a time, up to 64 rows a
// workgroup; a turn of the CUs costs 3 us and 1.65 or, in 64-column blocks, 1.25 a step.  (1 + q / 2 for all: 150 drawn products of 33 .. 128 rows
// take 0.94 of the time, but 31 of them, with outliers, give values 4e-4 .. 4e-3 of the root mean square from those of now.)
static int64_t one_bit_line(int64_t R, int nbc, int n, int batch)
{
    const int64_t z = (batch + 63) / 64;
    auto with = [&](int rg) {
        const int64_t tiles = (R + rg * 32 - 1) / (rg * 32) * z, jl = 8 / rg, steps = (nbc + jl - 1) / jl;
        const int64_t most = 256 / tiles < 32 ? 256 / tiles : 32;
        int64_t per_split = nbc;
        if (most > 1 && !(steps <= 4 && R * z * 64 > 1 << 18)) {
            const int64_t cols = (steps == 3 && most > 2 && R * z * 64 <= 1 << 17 ? 1 : ((steps + most - 1) / most + 1) / 2 * 2) * jl;
            if (cols < nbc) per_split = cols;
        }
        const int64_t n_split = (nbc + per_split - 1) / per_split;
        const int64_t pairs = ((per_split + jl - 1) / jl + 1) / 2, turns = (tiles * n_split + 255) / 256;
        int64_t cost = turns * (300 + pairs * 2 * (n == 128 ? 165 : 125));
        if (turns > 1 && rg == 2) cost += cost / 20;
        if (n_split > 1) cost += 200 + 20 * n_split + n_split * z * R / 160;   // the second launch and the partial sums
        return cost;
    };
    const int64_t a = with(4), b = with(2);
    return a < b ? a : b;
}
// of a launch of 33 .. 64 rows: by the line, whichever kernel then takes it
static bool fine_one_bit(const sbits_plan *plan, int64_t R, int nbc, int batch)
{
    return has_one_bit(plan) && few_rows(plan, R, nbc, batch).narrow * 100 < (double)(one_bit_line(R, nbc, plan->n, batch) + 250);
}
static bool takes_narrow(const sbits_plan *plan, int mat, const MpArgs &a)
{
    if (a.batch > 64 || a.ld_x > 1 << 25) return false;
    if (a.batch <= 32 && a.nbc <= MG_SPAN && a.R / 32 * ((a.batch + 15) / 16) <= 512) return true;
    const FewRows t = few_rows(plan, a.R, a.nbc, a.batch);
    if (a.batch <= 32) return t.narrow <= t.first;
    return t.narrow <= many_of(plan, mat, a.batch).us && (!has_one_bit(plan) || fine_one_bit(plan, a.R, a.nbc, a.batch));
}

// Rows of x the next launch takes of those that are left: 128 (two batch groups) while a group's byte offsets fit the 32 bits
// of a descriptor, else the 32 of the first kernel, whose addresses have 64.  65 .. 96 rows go as 64 and the rest where the kernels for
// few rows take the rest in less than the kernel of many rows takes longer for it (whose groups of 32 .. 64 rows make that rare), or by
// one_bit_line.
int sbits_mp_gemm_rows(const sbits_plan *plan, int mat, int64_t ld_x, int left)
{
    if (ld_x > 1 << 20) return left < 32 ? left : 32;
    if (left > 64 && left <= 96) {
        const int64_t R = plan->rows[mat];
        const int n = plan->n, nbc = (int)(plan->cols[mat] / n);
        const FewRows t = few_rows(plan, R, nbc, left - 64);
        const double rest = t.narrow < t.first ? t.narrow : t.first;
        if (has_one_bit(plan)) {
            if (one_bit_line(R, nbc, n, 64) + (int64_t)(rest * 100) + 300 <= one_bit_line(R, nbc, n, left)) return 64;
        } else if (many_of(plan, mat, 64).us + rest <= many_of(plan, mat, left).us) {
            return 64;
        }
    }
    return left < 128 ? left : 128;
}

// fine: rows of a product of more than 32, whose codes enter with the smaller offset in every kernel (1 bit in that of many rows by one_bit_line)
int sbits_launch_mp_gemm(sbits_plan *plan, int mat, const void *x_bf16, int64_t ld_x, int batch, bool fine,
                         const uint8_t *level, const int64_t *byte_off, const uint8_t *codes, const float *scale,
                         const float *zero, float *y, void *scratch)
{
    sbits_ctx *ctx = plan->ctx;
    MpArgs a;
    a.codes = codes; a.scale = scale; a.zero = zero; a.level = level; a.byte_off = byte_off;
    a.x = static_cast<const uint16_t *>(x_bf16);
    a.block_base = plan->base[mat]; a.ld_x = ld_x;
    a.R = (int)plan->rows[mat]; a.C = (int)plan->cols[mat]; a.m = plan->m; a.nbc = a.C / plan->n;
    a.batch = batch;
    for (int c = 0; c < sbits::MAX_CAND; ++c) a.bits[c] = c < plan->K ? plan->bits[c] : plan->bits[plan->K - 1];
    const bool one_bit = batch > 32 && batch <= 64 && fine_one_bit(plan, a.R, a.nbc, batch);
    if (takes_narrow(plan, mat, a)) {
        a.n_split = 1;
        a.out = y;
        // Workgroups of 16 waves while all of them are on the chip at once, one a CU (against 8 waves 2 .. 14 % faster): more codes
        // on their way; beyond that two workgroups of 8 waves, one of which computes while the other starts or ends (up to 25 %
        // faster).  x by way of LDS from 5 rows on: at 1 and 2 rows it costs 2 .. 6 %, at 3 and 4 it gives -2 .. 3, at 9 .. 16 3 .. 19, at 17
        // and more 3 .. 22 %.  The same sums all ways.
        const bool deep = a.R / 32 * ((batch + 15) / 16) <= sbits_cus(ctx);
        if (fine) {
            if (plan->n == 128) return deep ? launch_narrow<128, 16, true, true>(ctx, a) : launch_narrow<128, 8, true, true>(ctx, a);
            return deep ? launch_narrow<64, 16, true, true>(ctx, a) : launch_narrow<64, 8, true, true>(ctx, a);
        }
        if (batch > 4) {
            if (plan->n == 128) return deep ? launch_narrow<128, 16, false, true>(ctx, a) : launch_narrow<128, 8, false, true>(ctx, a);
            return deep ? launch_narrow<64, 16, false, true>(ctx, a) : launch_narrow<64, 8, false, true>(ctx, a);
        }
        if (plan->n == 128) return deep ? launch_narrow<128, 16, false, false>(ctx, a) : launch_narrow<128, 8, false, false>(ctx, a);
        return deep ? launch_narrow<64, 16, false, false>(ctx, a) : launch_narrow<64, 8, false, false>(ctx, a);
    }
    const bool many = batch > 32;
    const ManySplit ms = many ? many_of(plan, mat, batch) : ManySplit{0, 0, 0, 0.0};
    a.n_split = many ? ms.n_split : sbits_mp_gemm_splits(a.C, plan->n);
    a.out = a.n_split > 1 ? static_cast<float *>(scratch) : y;
    int rc;
    if (many) {
        if (one_bit) rc = plan->n == 128 ? launch_many_shape<128, true>(ctx, a, ms) : launch_many_shape<64, true>(ctx, a, ms);
        else rc = plan->n == 128 ? launch_many_shape<128, false>(ctx, a, ms) : launch_many_shape<64, false>(ctx, a, ms);
    } else {
        // Channels of a workgroup: x takes 32 .. 128 KiB of LDS, and as many waves as the registers allow (16) should be on a
        // CU.  64-column blocks up to 16 rows: four workgroups of 32 channels.  Else 64 (128 with 128 KiB of x), and half as
        // many where all workgroups are on the chip at once even so: 15872 x 2048 at 18 rows 11.5 -> 9.1 us with 64, 19584 x 896 at
        // 21 rows 9.4 -> 13.6; 2560 x 6784 at 2 rows 10.1 -> 9.3 with 32, 8096 x 7552 11.6 -> 14.1.  The same sums.
        const int cus = sbits_cus(ctx);
        const int64_t wgs32 = (int64_t)(a.R / 32) * a.n_split, wgs64 = (int64_t)((a.R + 63) / 64) * a.n_split;
        if (fine) {                                           // (the last rows of a large product: many workgroups)
            if (plan->n == 128) rc = batch <= 16 ? launch_mp<128, 1, 2, true>(ctx, a) : launch_mp<128, 2, 4, true>(ctx, a);
            else rc = batch <= 16 ? launch_mp<64, 1, 1, true>(ctx, a) : launch_mp<64, 2, 2, true>(ctx, a);
        } else if (plan->n == 128) {
            if (batch <= 16) rc = wgs32 <= 2 * cus ? launch_mp<128, 1, 1, false>(ctx, a) : launch_mp<128, 1, 2, false>(ctx, a);
            else rc = wgs64 <= cus ? launch_mp<128, 2, 2, false>(ctx, a) : launch_mp<128, 2, 4, false>(ctx, a);
        } else {
            if (batch <= 16) rc = launch_mp<64, 1, 1, false>(ctx, a);
            else rc = wgs32 <= cus ? launch_mp<64, 2, 1, false>(ctx, a) : launch_mp<64, 2, 2, false>(ctx, a);
        }
    }
    if (rc) return rc;
    if (a.n_split > 1) {
        const int64_t n = (int64_t)batch * a.R;
        hipLaunchKernelGGL(mp_gemm_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream,
                           (const float *)scratch, n, a.n_split, y);
        SBITS_HIP(ctx, hipGetLastError());
    }
    return SBITS_OK;
}
