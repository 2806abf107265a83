// Storage: byte offsets of the blocks and bit-packing of the chosen codes
// (one bitwidth per block, paper Sec. 5.3 "Inference Kernel").
//
// offsets : byte_off[i] = sum_{i' < i} m*n*c[level[i']]/8 (exclusive scan, int64).
// pack    : re-quantizes each block row at the block's bitwidth with the same
//           round-to-nearest grid as the cost table and writes the codes LSB
//           first: element e of the block (row-major) occupies bits
//           [e*c, (e+1)*c) of the block's little-endian bit stream.  A lane owns
//           8 consecutive weights = exactly c bytes of the stream; the lanes of
//           a row stage their bytes in LDS and the row is written out as dwords.
#include <string.h>

#include <mutex>

#include "pack_core.hpp"
#include "sbits_device.hpp"
#include "sbits_internal.hpp"

void sbits_fill_grid_consts(const int32_t *bits, int K, sbits::GridConsts *gc);

namespace sbits {

// ---- offsets --------------------------------------------------------------------
constexpr int OF_THREADS = 256;
constexpr int OF_ITEMS = 8;
constexpr int OF_TILE = OF_THREADS * OF_ITEMS;

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
struct BitsTab { int bits[MAX_CAND]; };
// (a level beyond the table, which no valid input holds, reads its last entry)
__device__ __forceinline__ int tab_bits(const BitsTab &bt, int lv) { return bt.bits[lv < MAX_CAND ? lv : MAX_CAND - 1]; }

__device__ __forceinline__ long long block_exclusive_scan(long long v, long long *total)
{
    __shared__ long long wsum[OF_THREADS / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    long long inc = v;
    for (int off = 1; off < 64; off <<= 1) {
        const long long t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    long long base = 0, tot = 0;
    for (int w = 0; w < OF_THREADS / 64; ++w) {
        if (w < wv) base += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

__global__ __launch_bounds__(OF_THREADS)
void tile_sum_kernel(const uint8_t *__restrict__ level, long long N, long long Mdiv8, BitsTab bt,
                     long long *__restrict__ tilesum, const unsigned *aborted)
{
    if (aborted && *aborted) return;                 // the levels are those of a search that gave up and is repeated
    const long long i0 = (long long)blockIdx.x * OF_TILE + (long long)threadIdx.x * OF_ITEMS;
    long long s = 0;
    for (int e = 0; e < OF_ITEMS; ++e)
        if (i0 + e < N) s += Mdiv8 * tab_bits(bt, level[i0 + e]);
    long long tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) tilesum[blockIdx.x] = tot;
}

// one workgroup: exclusive scan of the tile sums in place
__global__ __launch_bounds__(OF_THREADS)
void scan_tiles_kernel(long long *tilesum, long long ntiles)
{
    long long carry = 0;
    for (long long t0 = 0; t0 < ntiles; t0 += OF_THREADS) {
        const long long t = t0 + threadIdx.x;
        const long long v = t < ntiles ? tilesum[t] : 0;
        long long tot;
        const long long ex = block_exclusive_scan(v, &tot);
        if (t < ntiles) tilesum[t] = carry + ex;
        carry += tot;
    }
}

__global__ __launch_bounds__(OF_THREADS)
void tile_scan_kernel(const uint8_t *__restrict__ level, long long N, long long Mdiv8, BitsTab bt,
                      const long long *__restrict__ tilebase, int64_t *__restrict__ byte_off,
                      const unsigned *aborted)
{
    if (aborted && *aborted) return;
    const long long i0 = (long long)blockIdx.x * OF_TILE + (long long)threadIdx.x * OF_ITEMS;
    long long v[OF_ITEMS], s = 0;
    for (int e = 0; e < OF_ITEMS; ++e) {
        v[e] = (i0 + e < N) ? Mdiv8 * tab_bits(bt, level[i0 + e]) : 0;
        s += v[e];
    }
    long long tot;
    long long acc = tilebase[blockIdx.x] + block_exclusive_scan(s, &tot);
    for (int e = 0; e < OF_ITEMS; ++e) {
        if (i0 + e < N) byte_off[i0 + e] = acc;
        acc += v[e];
        if (i0 + e == N - 1) byte_off[N] = acc;
    }
}

// All in one launch, because a launch costs 4.6 us: a workgroup adds up all levels before its tile by itself, 16 a load, four at a
// time through a byte permute that looks their bitwidths up.  One launch against three, calls one behind the other: 1 k blocks
// 3.7 and 8.5 us, 33 k 7.4 and 9.7, 106 k 8.8 and 9.8, 197 k 9.9 and 10.2, 262 k 10.8 and 10.4, 426 k 13.3 and 11.1, 1 M 22.4 and
// 15.5: the last workgroup reads all levels, so the line is where that takes what two launches do.
constexpr int OO_THREADS = 1024, OO_TILE = OO_THREADS * OF_ITEMS;
constexpr int64_t OO_MAX_BLOCKS = 3 << 16;
__global__ __launch_bounds__(OO_THREADS)
void offsets_kernel(const uint8_t *__restrict__ level, int N, long long Mdiv8, BitsTab bt, int64_t *__restrict__ byte_off,
                    const unsigned *aborted)
{
    __shared__ unsigned bits_before;
    __shared__ int wave_bits[OO_THREADS / 64];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, t0 = (int)blockIdx.x * OO_TILE;
    const unsigned stop = aborted ? *aborted : 0u;   // nonzero: the levels are those of a search that gave up and is repeated
    if (tid == 0) bits_before = 0u;
    unsigned lo = 0u, hi = 0u;                       // bitwidths of levels 0 .. 3, 4 .. 7
#pragma unroll
    for (int l = 0; l < 4; ++l) { lo |= (unsigned)bt.bits[l] << (8 * l); hi |= (unsigned)bt.bits[l + 4] << (8 * l); }
    unsigned before = 0u;                            // (OO_MAX_BLOCKS blocks of at most 8 bits: far below 2^32)
    const int i0 = t0 + tid * OF_ITEMS;
    u32x2_t own = {0u, 0u};
    if (i0 + OF_ITEMS <= N) __builtin_memcpy(&own, level + i0, 8);
    for (int j0 = tid * 16; j0 < t0; j0 += 4 * OO_THREADS * 16) {    // (t0 is a multiple of 16; all loads of a turn before any use)
        u32x4_t v[4];
        unsigned any = 0u;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int j = j0 + b * OO_THREADS * 16;
            v[b] = u32x4_t{0u, 0u, 0u, 0u};
            if (j < t0) __builtin_memcpy(&v[b], level + j, 16);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) any |= v[b].x | v[b].y | v[b].z | v[b].w;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (j0 + b * OO_THREADS * 16 >= t0) continue;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if ((any & 0xf8f8f8f8u) == 0u) {
                    before = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(hi, lo, v[b][w]), 0u, before);
                } else {
                    for (int e = 0; e < 4; ++e) before += (unsigned)tab_bits(bt, (int)(v[b][w] >> (8 * e) & 255u));
                }
            }
        }
    }
    int v[OF_ITEMS], s = 0;
#pragma unroll
    for (int e = 0; e < OF_ITEMS; ++e) {
        int lv = (int)((e < 4 ? own.x : own.y) >> (8 * (e & 3)) & 255u);
        if (i0 + OF_ITEMS > N && i0 + e < N) lv = level[i0 + e];     // (the last blocks)
        v[e] = i0 + e < N ? tab_bits(bt, lv) : 0;
        s += v[e];
    }
    int inc = s;
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == 63) wave_bits[wave] = inc;
    for (int off = 32; off; off >>= 1) before += __shfl_xor(before, off);
    __syncthreads();
    if (stop) return;
    if (lane == 0 && before) atomicAdd(&bits_before, before);
    __syncthreads();
    int base = inc - s;
#pragma unroll
    for (int w = 0; w < OO_THREADS / 64; ++w) base += w < wave ? wave_bits[w] : 0;
    long long acc = Mdiv8 * ((long long)bits_before + base);
#pragma unroll
    for (int e = 0; e < OF_ITEMS; ++e) {
        if (i0 + e < N) byte_off[i0 + e] = acc;
        acc += Mdiv8 * v[e];
        if (i0 + e == N - 1) byte_off[N] = acc;
    }
}

// ---- pack -------------------------------------------------------------------------
constexpr int PK_THREADS = 256;

// Geometry as in the cost kernel: the GW = 64/LPG lane groups of a wave sit on BX adjacent
// blocks of one block row (contiguous reads), the four waves (and the remaining OW groups of a
// wave) take different octets.  A workgroup is one step of one unit; each lane group packs one
// octet (8 rows) of one block, staged in LDS and written out as one contiguous run.  Weights pass the caches by (non-temporal: 5 to 8 %
// whatever the block width) unless CACHED, see caches_weights(); scale and zero of the octet leave in one store each (64 columns: 20 %).  Codes are non-temporal where a
// group's store covers whole lines, from 256 columns (2 to 5 %); narrower blocks put lines together from several stores, which is the
// caches' work (16384 x 16384 at 0 to 8 bits, 128-row blocks: 16 columns 213 us, non-temporal 534; 32 columns 175 and 298, 64 124 and
// 145, 128 115 and 118).  Two 8B-shaped layers in 256-column blocks 241 -> 182 us in all.
template <int LPG>
struct PackGeom {
    static constexpr int GW = 64 / LPG;
    static constexpr int BX = GW < 8 ? GW : 8;
    static constexpr int OW = GW / BX;
    static constexpr int OS = 4 * OW;
    static int blocks_per_unit(int m) { const int opb = m / 8; return opb >= OS ? BX : BX * (OS / opb); }
    static int steps(int m) { const int opb = m / 8; return opb >= OS ? opb / OS : 1; }
};

template <int LPG, bool CACHED>
__global__ __launch_bounds__(PK_THREADS)
void pack_kernel(const MatDesc *__restrict__ descs, MatDesc one, const int *__restrict__ wg_start, int n_mats,
                 const uint16_t *__restrict__ W, int m, const uint8_t *__restrict__ level,
                 const int64_t *__restrict__ byte_off, uint8_t *__restrict__ codes, float *__restrict__ scale,
                 float *__restrict__ zero, GridConsts gc, const unsigned *aborted)
{
    if (aborted && *aborted) return;                 // the levels are those of a search that gave up and is repeated
    using G = PackGeom<LPG>;
    constexpr int BX = G::BX, OS = G::OS, NG = PK_THREADS / LPG;
    __shared__ __align__(16) uint8_t stage[NG][8 * LPG * 8];     // per group: 8 rows x LPG*c bytes (c <= 8)

    const int mat = descs ? find_matrix(wg_start, n_mats, (int)blockIdx.x) : 0;
    const MatDesc d = descs ? descs[mat] : one;
    const int lid = (int)blockIdx.x - (descs ? wg_start[mat] : 0);
    const int opb = m >> 3;
    const int bpu = opb >= OS ? BX : BX * (OS / opb);
    const int steps = opb >= OS ? opb / OS : 1;
    const int upr = (d.nbc + bpu - 1) / bpu;
    const int I = lid / (upr * steps);
    const int rem = lid - I * (upr * steps);
    const int U = rem / steps, p = rem - U * steps;

    const int tid = threadIdx.x;
    const int lig = tid % LPG;
    const int g = tid / LPG;
    const int gw = (tid & 63) / LPG;
    const int slot = (tid >> 6) * G::OW + gw / BX;
    const int bl = (gw % BX) + (opb >= OS ? 0 : BX * (slot / opb));
    const int o = (opb >= OS ? slot : slot % opb) + p * OS;
    const int J = U * bpu + bl;
    const bool valid = J < d.nbc;
    const int Jc = valid ? J : d.nbc - 1;
    const int64_t gb = d.block_base + (int64_t)I * d.nbc + Jc;   // global block id
    const LevelConsts lk = level_consts(gc, level[gb]);
    const int c = lk.c;

    const uint16_t *__restrict__ src = W + d.elem_off + ((int64_t)I * m + (int64_t)o * 8) * d.cols +
                                       (int64_t)Jc * (LPG * 8) + lig * 8;
    uint4 raw[8];
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
        const __attribute__((address_space(1))) u32x4_t *const p = (const __attribute__((address_space(1))) u32x4_t *)(src + (int64_t)rr * d.cols);
        u32x4_t v;
        if constexpr (CACHED) v = *p;
        else v = __builtin_nontemporal_load(p);
        raw[rr] = make_uint4(v.x, v.y, v.z, v.w);
    }

    const int row_bytes = LPG * c;
    float keep_s = 0.0f, keep_z = 0.0f;              // row lig's
    const bool odd = (lig & 1) != 0;                 // even lanes divide qmax/R, odd lanes R/qmax
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
        float scl, mn;
        const unsigned long long word = quant_pack_row<LPG>(raw[rr], lk, odd, scl, mn);
        uint8_t *mine = &stage[g][rr * row_bytes + lig * c];
        store_code_bytes(mine, word, c);
        if constexpr (LPG >= 8) {
            keep_s = lig == rr ? scl : keep_s;
            keep_z = lig == rr ? mn + 0.0f : keep_z;
        } else if (valid && lig == 0) {
            const int64_t ri = gb * m + o * 8 + rr;
            scale[ri] = scl;
            zero[ri] = mn + 0.0f;
        }
    }
    if (LPG >= 8 && valid && lig < 8) {              // the octet's eight rows in one store
        const int64_t ri = gb * m + o * 8 + lig;
        scale[ri] = keep_s;
        zero[ri] = keep_z;
    }
    __syncthreads();
    if (valid) {
        // the octet's 8 rows are consecutive in the block's stream: one run of 8*row_bytes bytes
        uint8_t *dst = codes + byte_off[gb] + (int64_t)o * 8 * row_bytes;
        const int nbytes = 8 * row_bytes;            // a multiple of 8
        const uint32_t *s32 = reinterpret_cast<const uint32_t *>(&stage[g][0]);
        uint32_t *d32 = reinterpret_cast<uint32_t *>(dst);
        for (int k = lig; k < nbytes / 4; k += LPG) {
            if constexpr (LPG >= 32) __builtin_nontemporal_store(s32[k], (__attribute__((address_space(1))) uint32_t *)d32 + k);
            else d32[k] = s32[k];
        }
    }
}

struct PackLaunch {
    const MatDesc *descs;
    MatDesc one;
    const int *wg_start;
    int n_mats;
    int64_t total_wg;
    const uint16_t *W;
    bool cached;
    int m;
    const uint8_t *level;
    const int64_t *byte_off;
    uint8_t *codes;
    float *scale, *zero;
    GridConsts gc;
    const unsigned *aborted;
};

// Ordinary loads where weights that a program packs again and again, with other levels each time, stay in the 256 MiB memory-side cache
// beside their codes, which non-temporal loads read past in blocks of up to 64 columns.  Packed again, ordinary / non-temporal: 8 columns
// 20 MiB 20.0 us and 20.4, 28 22.8 and 24.4, 80 47.4 and 56.4, 150 112 and 100; 16 columns 36 MiB 23.5 and 25.2, 170 56 and 69, 190 100 and 97; 32
// columns 44 MiB 23.2 and 26.4, 170 48.6 and 62.9, 215 84 and 82; 64 columns 60 MiB 24.3 and 23.8, 110 41.1 and 47.8, 215 64.2 and 64.3.  From
// 128 columns on they gain little.  Just after the copies were made both take the same from 60 MiB on.  Not in a search: there they
// cost more (32 columns, 16864 x 3104: 445 us and, with ordinary loads, 456; 32 searches of 60 .. 180 MiB 1.2 % on average).
static bool caches_weights(int n, int64_t weights)
{
    const int64_t mib = weights * 2 >> 20;
    return n <= 64 && mib > (n == 8 ? 24 : n < 64 ? 40 : 72) && mib <= (n == 8 ? 144 : n == 16 ? 176 : 208);
}

template <int LPG>
static int launch_pack_l(sbits_ctx *ctx, const PackLaunch &a)
{
    if (a.total_wg > 0x7fffffff) return SBITS_ERR_BAD_SHAPE;
    if (a.total_wg == 0) return SBITS_OK;
    auto *fn = &pack_kernel<LPG, false>;
    if constexpr (LPG <= 8) {
        if (a.cached) fn = &pack_kernel<LPG, true>;
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)a.total_wg), dim3(PK_THREADS), 0, ctx->stream,
                       a.descs, a.one, a.wg_start, a.n_mats, a.W, a.m, a.level, a.byte_off, a.codes, a.scale,
                       a.zero, a.gc, a.aborted);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

static int launch_pack(int n, sbits_ctx *ctx, const PackLaunch &a)
{
    switch (n / 8) {
    case 1:  return launch_pack_l<1>(ctx, a);
    case 2:  return launch_pack_l<2>(ctx, a);
    case 4:  return launch_pack_l<4>(ctx, a);
    case 8:  return launch_pack_l<8>(ctx, a);
    case 16: return launch_pack_l<16>(ctx, a);
    case 32: return launch_pack_l<32>(ctx, a);
    case 64: return launch_pack_l<64>(ctx, a);
    }
    return SBITS_ERR_BAD_SHAPE;
}

static int64_t pack_wgs(int m, int n, int nbr, int nbc)
{
    int bpu = 1, st = 1;
    switch (n / 8) {
    case 1:  bpu = PackGeom<1>::blocks_per_unit(m);  st = PackGeom<1>::steps(m); break;
    case 2:  bpu = PackGeom<2>::blocks_per_unit(m);  st = PackGeom<2>::steps(m); break;
    case 4:  bpu = PackGeom<4>::blocks_per_unit(m);  st = PackGeom<4>::steps(m); break;
    case 8:  bpu = PackGeom<8>::blocks_per_unit(m);  st = PackGeom<8>::steps(m); break;
    case 16: bpu = PackGeom<16>::blocks_per_unit(m); st = PackGeom<16>::steps(m); break;
    case 32: bpu = PackGeom<32>::blocks_per_unit(m); st = PackGeom<32>::steps(m); break;
    case 64: bpu = PackGeom<64>::blocks_per_unit(m); st = PackGeom<64>::steps(m); break;
    }
    return (int64_t)nbr * ((nbc + bpu - 1) / bpu) * st;
}

}  // namespace sbits

using namespace sbits;

size_t sbits_offsets_ws_bytes(int64_t N)
{
    const int64_t ntiles = (N + OF_TILE - 1) / OF_TILE;
    return sbits_align_up((size_t)ntiles * 8, 256);
}

// ---- offsets without a caller workspace ---------------------------------------------
// The tile sums of the scan in a fixed device array instead of the caller's workspace, for
// callers that cannot allocate one.  Each GPU holds its own copy of the array at its own
// address; the address is looked up once per device (with that device current) and kept.
static __device__ __align__(256) long long scratch[SBITS_OFFSETS_STATIC_MAX_BLOCKS / OF_TILE];
static_assert(SBITS_OFFSETS_STATIC_MAX_BLOCKS % OF_TILE == 0, "whole tiles");

constexpr int OF_MAX_DEVICES = 64;
static std::mutex g_scratch_lock;
static long long *g_scratch_ptr[OF_MAX_DEVICES];     // device address of scratch[], per device ordinal

// Device address of this GPU's scratch array (ctx->device must be the current device).
int sbits_offsets_static_setup(sbits_ctx *ctx)
{
    if (ctx->device < 0 || ctx->device >= OF_MAX_DEVICES) return SBITS_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[ctx->device]) {
        long long *ptr = nullptr;
        SBITS_HIP(ctx, hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)));
        if (!ptr) return SBITS_ERR_HIP;
        g_scratch_ptr[ctx->device] = ptr;
    }
    return SBITS_OK;
}

int sbits_launch_offsets_static(sbits_ctx *ctx, const uint8_t *level, int64_t N, int m, int n,
                                const int32_t *bits, int K, int64_t *byte_off)
{
    if (N > SBITS_OFFSETS_STATIC_MAX_BLOCKS) return SBITS_ERR_WORKSPACE;
    if (ctx->device < 0 || ctx->device >= OF_MAX_DEVICES) return SBITS_ERR_HIP;
    long long *ptr;
    {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        ptr = g_scratch_ptr[ctx->device];
    }
    if (!ptr) return SBITS_ERR_HIP;                  // sbits_create resolves it; never the array's host-side name
    // every tile sum in use is written by the first kernel before the others read it: nothing to clear
    return sbits_launch_offsets(ctx, level, N, m, n, bits, K, byte_off, ptr);
}

int sbits_launch_offsets(sbits_ctx *ctx, const uint8_t *level, int64_t N, int m, int n,
                         const int32_t *bits, int K, int64_t *byte_off, void *ws, const unsigned *aborted)
{
    BitsTab bt;
    for (int c = 0; c < sbits::MAX_CAND; ++c) bt.bits[c] = c < K ? bits[c] : bits[K - 1];
    const long long Mdiv8 = (long long)m * n / 8;
    if (N <= OO_MAX_BLOCKS) {
        hipLaunchKernelGGL(offsets_kernel, dim3((unsigned)((N + OO_TILE - 1) / OO_TILE)), dim3(OO_THREADS), 0, ctx->stream, level, (int)N,
                           Mdiv8, bt, byte_off, aborted);
        SBITS_HIP(ctx, hipGetLastError());
        return SBITS_OK;
    }
    const int64_t ntiles = (N + OF_TILE - 1) / OF_TILE;
    long long *tiles = static_cast<long long *>(ws);
    hipLaunchKernelGGL(tile_sum_kernel, dim3((unsigned)ntiles), dim3(OF_THREADS), 0, ctx->stream,
                       level, (long long)N, Mdiv8, bt, tiles, aborted);
    hipLaunchKernelGGL(scan_tiles_kernel, dim3(1), dim3(OF_THREADS), 0, ctx->stream, tiles, (long long)ntiles);
    hipLaunchKernelGGL(tile_scan_kernel, dim3((unsigned)ntiles), dim3(OF_THREADS), 0, ctx->stream,
                       level, (long long)N, Mdiv8, bt, tiles, byte_off, aborted);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

int sbits_launch_pack(sbits_ctx *ctx, const void *Wp, int64_t R, int64_t C, int m, int n,
                      const int32_t *bits, int K, const uint8_t *level, const int64_t *byte_off,
                      int64_t block_base, uint8_t *codes, float *scale, float *zero)
{
    PackLaunch a;
    memset(&a, 0, sizeof a);
    sbits_fill_grid_consts(bits, K, &a.gc);
    a.one.rows = R; a.one.cols = C; a.one.nbr = (int)(R / m); a.one.nbc = (int)(C / n);
    a.one.block_base = block_base;
    a.n_mats = 1;
    a.total_wg = pack_wgs(m, n, a.one.nbr, a.one.nbc);
    a.W = static_cast<const uint16_t *>(Wp);
    a.cached = caches_weights(n, R * C);
    a.m = m;
    a.level = level; a.byte_off = byte_off; a.codes = codes; a.scale = scale; a.zero = zero;
    return launch_pack(n, ctx, a);
}

// workgroups per matrix, summed up
void sbits_pack_tables(sbits_plan *plan)
{
    int64_t tot = 0;
    for (int i = 0; i < plan->n_mats; ++i) {
        plan->pack_wg_start.push_back((int)tot);
        tot += pack_wgs(plan->m, plan->n, plan->descs[i].nbr, plan->descs[i].nbc);
        if (tot > 0x7fffffff) { plan->pack_wg_start.clear(); return; }
    }
    plan->pack_wg_start.push_back((int)tot);
}

// all matrices of the plan in one launch; the descriptor table is already in the workspace head.  again: see caches_weights
int sbits_launch_pack_all(sbits_plan *plan, const void *w_re, const uint8_t *level, const int64_t *byte_off,
                          uint8_t *codes, float *scale, float *zero, bool again, void *ws, const unsigned *aborted)
{
    sbits_ctx *ctx = plan->ctx;
    PackLaunch a;
    memset(&a, 0, sizeof a);
    a.aborted = aborted;
    sbits_fill_grid_consts(plan->bits, plan->K, &a.gc);
    if (plan->pack_wg_start.empty()) return SBITS_ERR_BAD_SHAPE;
    a.descs = sbits_desc_ptr(ws);
    a.wg_start = sbits_prefix_ptr(plan, ws, SLOT_PACK_WGS);
    a.n_mats = plan->n_mats;
    a.total_wg = plan->pack_wg_start.back();
    a.W = static_cast<const uint16_t *>(w_re);
    a.cached = again && caches_weights(plan->n, plan->sum_elems);
    a.m = plan->m;
    a.level = level; a.byte_off = byte_off; a.codes = codes; a.scale = scale; a.zero = zero;
    return launch_pack(plan->n, ctx, a);
}
