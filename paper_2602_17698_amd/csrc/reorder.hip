// Bi-directional channel reordering (paper Sec. 4.1): channel scores, argsort,
// and the reorder-gather of weights and sensitivities.  Every kernel serves all
// matrices of a plan in one launch (descriptor table + workgroup prefix) or a
// single matrix whose descriptor travels as a kernel argument.
//
// Scores.  Row score = l1 norm of the row of S, column score = l1 norm of the
// column, each summed in the canonical order: runs of 8 consecutive elements
// left to right from +0, then an adjacent-pair tree over the runs (zero padded
// to a power of two).  One pass over S serves both directions.  A workgroup of
// four waves walks a band of up to 512 rows over a panel of 4096 columns, row by row
// (16 KiB of consecutive bytes per row).  The partial trees (per row and panel; per column
// and band) go to the workspace and a small kernel finishes them.
//
// Argsort.  Descending by score, ties to the lower index: inverted ordered-float
// keys with the index behind them, sorted in chunks of 1024; what an array has
// of chunks is merged by rank.  All arrays of the plan side by side.
//
// Gather.  out[i][j] = in[rp[i]][cp[j]]: the source row is staged in LDS with
// coalesced 128-bit loads and read out permuted, so global traffic stays
// coalesced in both directions.
#include <string.h>

#include <vector>

#include "sbits_device.hpp"
#include "sbits_internal.hpp"

namespace sbits {

// ================================================================ scores
constexpr int SC_THREADS = 256;
constexpr int SC_ROWS = 512;    // most rows per band (64 octets): one workgroup walks a whole band
constexpr int SC_COLS = 512;    // columns per segment: one wave, two 1 KiB loads per row
constexpr int SC_PANEL = 8;     // segments per workgroup: 4 waves x 2 segments = 4096 columns = 16 KiB per row

// rowpart[r][panel] : tree over the 8 segments' trees over their 64 column runs (zero beyond C)
// colpart[band][c]  : tree over the row runs (8 rows each) of band (zero beyond R)
//
// A workgroup reads rows of 16 KiB (its panel of 8 segments) top to bottom; wave w owns segments w and w + 4, and of each row
// brings four contiguous KiB of its own, non-temporal, straight into a ring of rows in LDS: no barrier, no registers
// for what is on its way.  A lane reads the 8 columns of a run of each segment out of it; a row's runs go through a
// butterfly over the wave, column sums stay in registers for the whole band (16 columns a lane, an adjacent-pair tree over
// its octets).
// What bounds it is HBM, and what keeps it from the 7.0 TB/s of loads alone is writing: a few isolated writes cost the stream
// of reads far more than their bytes (28 GB in 4.03 ms without any, 4.71 with a partial sum per 512 and per 256 elements, 0.6 % of the
// bytes).  So a row's 8 segments are added up before they leave, bands have 512 rows where there are many, and what is
// written goes through the L2 at once (sc1: 4.71 -> 4.36 ms, nontemporal 4.41).  All together 4.71 -> 4.21 ms (6.6 TB/s); four layers of that
// model 600 -> 527 us, two 283 -> 264, one 144 -> 128, 8192 x 28672 four times 640 -> 547, 2048 x 2048 10.5 -> 8.2.  Its predecessor held the
// rows on their way in registers.
// A band has band_rows rows, a power of two: see sbits_score_rows().
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// RING: rows of a wave on their way.  3 where two workgroups with the row sums of 512 rows share a CU, 4 with 256 rows or fewer, 8 where a CU has one.
template <int RING>
__global__ __launch_bounds__(SC_THREADS, 2)
void score_partial_kernel(const MatDesc *__restrict__ descs, MatDesc one, const int *__restrict__ wg_start,
                          int n_mats, int band_rows, float *__restrict__ rowpart_all, float *__restrict__ colpart_all)
{
    constexpr int ROW = 2 * SC_COLS * 4;                 // bytes of a wave's part of a row
    extern __shared__ __attribute__((aligned(1024))) unsigned char ring[];        // [wave][slot], and the band's row sums [row][segment of the panel]
    float *const rowsum = reinterpret_cast<float *>(ring + SC_THREADS / 64 * RING * ROW);
    const int mat = descs ? __builtin_amdgcn_readfirstlane(find_matrix(wg_start, n_mats, (int)blockIdx.x)) : 0;
    const MatDesc &d = descs ? descs[mat] : one;
    const int lid = (int)blockIdx.x - (descs ? wg_start[mat] : 0);
    // (uniform, which the compiler does not see where they come through a pointer)
    auto uniform = [](int64_t v) {
        return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32)) << 32 |
                         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v));
    };
    const int npanel = __builtin_amdgcn_readfirstlane(d.npanel);
    const int band = __builtin_amdgcn_readfirstlane(lid / npanel), panel = __builtin_amdgcn_readfirstlane(lid - band * npanel);
    const int R = (int)uniform(d.rows), C = (int)uniform(d.cols);
    float *__restrict__ rowpart = rowpart_all + uniform(d.rowpart_off);
    float *__restrict__ colpart = colpart_all + uniform(d.colpart_off);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int seg0 = panel * SC_PANEL + wave;            // and seg0 + 4
    const int rbase = band * band_rows;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring + (uint32_t)(wave * RING * ROW);

    const uint32_t rowsum0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring + (uint32_t)(SC_THREADS / 64 * RING * ROW);
    // row r of the band into a slot of the ring; what is past the matrix's columns or rows reads as zero and is not fetched
    const int64_t pitch = uniform(d.ld_s) * 4;
    const char *const S = reinterpret_cast<const char *>(uniform((int64_t)(uintptr_t)d.s)) + (int64_t)rbase * pitch;
    const int rows = min(band_rows, R - rbase);
    auto fetch = [&](int r, uint32_t slot) {
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(S) + r * pitch, 0, r < rows ? C * 4 : 0, 0x00027000);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(slot + (uint32_t)q * 1024), 16,
                                                     (seg0 + 4 * (q >> 1)) * (SC_COLS * 4) + (q & 1) * 1024 + lane * 16, 0, 0, 2 /* nontemporal */);
    };

    constexpr int SC_THROUGH = 16;                       // sc1
    const rsrc_t cols_out = __builtin_amdgcn_make_buffer_rsrc(colpart + (int64_t)band * C, 0, C * 4, 0x00027000);
    const rsrc_t rows_out = __builtin_amdgcn_make_buffer_rsrc(rowpart + (int64_t)rbase * npanel + panel, 0, ((rows - 1) * npanel + 1) * 4, 0x00027000);
    float colrun[16], t1[16], t2[16], t3[16], t4[16], t5[16], t6[16];
    uint32_t slot = lds0;
    const uint32_t last = lds0 + (RING - 1) * ROW;
#pragma unroll
    for (int r = 0; r < RING; ++r) fetch(r, lds0 + (uint32_t)(r * ROW));
#pragma unroll 1
    for (int oc = 0; oc < band_rows / 8; ++oc) {
        float keep = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            f32x4_t v[2][2];
            // the row is there (those behind it may be on their way; a store in between makes the wait longer, never shorter)
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * (RING - 1)) : "memory");
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:16\n\tds_read_b128 %2, %4 offset:2048\n\t"
                         "ds_read_b128 %3, %4 offset:2064\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(v[0][0]), "=&v"(v[0][1]), "=&v"(v[1][0]), "=&v"(v[1][1]) : "v"(slot + (uint32_t)lane * 32) : "memory");
            fetch(8 * oc + k + RING, slot);
            slot = slot == last ? lds0 : slot + ROW;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    x[e] = fabsf(v[j][e >> 2][e & 3]);
                    colrun[j * 8 + e] = (k == 0 ? 0.0f : colrun[j * 8 + e]) + x[e];       // top to bottom, 8 rows
                }
                float rs = x[0];                              // a run of 8, left to right
#pragma unroll
                for (int e = 1; e < 8; ++e) rs = rs + x[e];
                rs = group_allreduce<64>(rs, OpAdd());           // the adjacent-pair tree over the segment's 64 runs
                keep = lane == 8 * j + k ? rs : keep;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) asm volatile("" : "+v"(colrun[e]));      // (now, not all rows' at the octet's end, which spills)
        }
        // (asm: the compiler would wait for the rows on their way before it touches LDS)
        if (lane < 16)
            asm volatile("ds_write_b32 %0, %1" :: "v"(rowsum0 + (uint32_t)(((8 * oc + (lane & 7)) * SC_PANEL + wave + 4 * (lane >> 3)) * 4)), "v"(keep) : "memory");
        // columns: adjacent-pair tree over the band's octets, fed one octet at a time
        auto add = [&](const float (&t)[16]) {
#pragma unroll
            for (int e = 0; e < 16; ++e) colrun[e] = t[e] + colrun[e];
        };
        auto set = [&](float (&t)[16]) {
#pragma unroll
            for (int e = 0; e < 16; ++e) t[e] = colrun[e];
        };
        if (oc & 1) {
            add(t1);
            if (oc & 2) {
                add(t2);
                if (oc & 4) {
                    add(t3);
                    if (oc & 8) {
                        add(t4);
                        if (oc & 16) {
                            add(t5);
                            if (oc & 32) add(t6);
                            else set(t6);
                        } else set(t5);
                    } else set(t4);
                } else set(t3);
            } else set(t2);
        } else set(t1);
        if (oc == band_rows / 8 - 1) {                        // (all the octets, a power of two: the tree's root)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int c = (seg0 + 4 * j) * SC_COLS + lane * 8;
                if (c >= C) continue;                         // (a run is inside or past the matrix)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4_t v;
                    v.x = __float_as_uint(colrun[j * 8 + h * 4]); v.y = __float_as_uint(colrun[j * 8 + h * 4 + 1]);
                    v.z = __float_as_uint(colrun[j * 8 + h * 4 + 2]); v.w = __float_as_uint(colrun[j * 8 + h * 4 + 3]);
                    __builtin_amdgcn_raw_buffer_store_b128(v, cols_out, (c + 4 * h) * 4, 0, SC_THROUGH);
                }
            }
        }
    }
    // the panel's segments of a row: the next three levels of its tree
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    for (int r = threadIdx.x; r < rows; r += SC_THREADS) {
        const float *const x = rowsum + r * SC_PANEL;
        const float v = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rows_out, r * npanel * 4, 0, SC_THROUGH);
    }
}

// adjacent-pair tree over 32 leaves x[(i0 + i) * stride], i < 32, zero beyond n
__device__ __forceinline__ float tree32(const float *__restrict__ x, int i0, int n, int64_t stride)
{
    float v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = (i0 + i < n) ? x[(int64_t)(i0 + i) * stride] : 0.0f;
#pragma unroll
    for (int w = 16; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) v[i] = v[2 * i] + v[2 * i + 1];
    return v[0];
}

// adjacent-pair tree over n <= 128 leaves, zero padded to a power of two (adding the padding
// is the identity, so trees of 32, 64 and 128 leaves nest)
__device__ __forceinline__ float tree_upto128(const float *__restrict__ x, int n, int64_t stride)
{
    float a = tree32(x, 0, n, stride);
    if (n > 32) a = a + tree32(x, 32, n, stride);
    if (n > 64) {
        float b = tree32(x, 64, n, stride);
        if (n > 96) b = b + tree32(x, 96, n, stride);
        a = a + b;
    }
    return a;
}

// one thread per channel; scores = [rows of matrix 0 | rows of matrix 1 | ... | cols of matrix 0 | ...]
__global__ void score_finish_kernel(const MatDesc *__restrict__ descs, MatDesc one, int n_mats,
                                    int64_t sum_rows, int64_t sum_cols,
                                    const float *__restrict__ rowpart_all, const float *__restrict__ colpart_all,
                                    float *__restrict__ rs_all, float *__restrict__ cs_all)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= sum_rows + sum_cols) return;
    const bool is_row = t < sum_rows;
    const int64_t ch = is_row ? t : t - sum_rows;
    int mat = 0;
    if (descs) {                                     // largest mat with offset <= ch
        int lo = 0, hi = n_mats;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            const int64_t o = is_row ? descs[mid].row_off : descs[mid].col_off;
            if (o <= ch) lo = mid; else hi = mid;
        }
        mat = lo;
    }
    const MatDesc &d = descs ? descs[mat] : one;
    if (is_row) {
        const int64_t r = ch - d.row_off;
        rs_all[ch] = tree_upto128(rowpart_all + d.rowpart_off + r * d.npanel, d.npanel, 1);
    } else {
        const int64_t c = ch - d.col_off;
        cs_all[ch] = tree_upto128(colpart_all + d.colpart_off + c, d.nband, d.cols);
    }
}

// ================================================================ argsort
// Bound by the latency of a chain of dependent steps, not by memory, so the chain is cut short: chunks of 1024 channels are
// sorted side by side, a lane per channel (bitonic network: 45 steps inside the wave, 10 through LDS), and the rank of a
// channel in its array is its place in its own chunk plus, for every other chunk, the number of keys there that go before
// it (binary search in LDS, all the chunks of the array).  A layer with arrays of up to 28672 channels: 42 us, where one
// workgroup an array with four radix passes took 242; up to 14336: 22 (104); 512, the chunk sort alone: 6.7 (10.7).
constexpr int CS_LEN = 1024, CS_THREADS = CS_LEN;             // channels of a chunk, one a thread
constexpr int RK_THREADS = 512;                               // of the ranking: half a chunk, so that more CUs share an array

__device__ __forceinline__ unsigned int sort_key(float f)
{
    const unsigned int u = __float_as_uint(f + 0.0f);                 // -0 -> +0
    const unsigned int ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);   // ascending in f
    return ~ord;                                                      // ascending key = descending score
}

// Array a of the launch: a < n_mats -> the rows of matrix a, else the columns of matrix a - n_mats.
// arr_mode (may be null = all SORT): what to do with array a; arr_segment (with arr_mode): 0 or the
// length of the pieces that are sorted one by one (a permutation that stays inside attention heads).
enum { ARR_SORT = 0, ARR_IDENTITY = 1, ARR_SKIP = 2 };

struct SortArrays {
    const MatDesc *descs;
    MatDesc one;
    int n_mats, per;                                          // workgroups per array: they take its chunks in turn
    int64_t sum_rows;
    const int *mode, *segment;
    int32_t *row_perm, *col_perm;
};
struct SortArray {
    int n, piece, mode;                                       // channels, channels per piece
    int64_t off;                                              // of its scores, keys and indices
    int32_t *perm;
};
__device__ __forceinline__ SortArray sort_array(const SortArrays &s, int a)
{
    const bool is_row = a < s.n_mats;
    const MatDesc &d = s.descs ? s.descs[is_row ? a : a - s.n_mats] : s.one;
    SortArray o;
    o.n = (int)(is_row ? d.rows : d.cols);
    o.off = is_row ? d.row_off : s.sum_rows + d.col_off;
    o.perm = is_row ? s.row_perm + d.row_off : s.col_perm + d.col_off;
    o.mode = s.mode ? s.mode[a] : ARR_SORT;
    o.piece = (s.mode && s.segment[a] > 0) ? s.segment[a] : o.n;
    return o;
}

// x of lane ^ J
template <int J>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t x)
{
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_XOR1, 0xf, 0xf, true);
    else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_XOR2, 0xf, 0xf, true);
    else if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, true);   // row_ror:8
    else if constexpr (J < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, J << 10 | 0x1f);
    else return (uint32_t)__shfl_xor((int)x, J);
}

// one step of the network: the thread keeps the smaller or the larger of its key and thread (tid ^ J)'s
template <int K, int J>
__device__ __forceinline__ void sort_step(uint64_t &x, int tid, uint64_t (*buf)[CS_LEN], int &turn)
{
    uint64_t y;
    if constexpr (J >= 64) {
        buf[turn][tid] = x;
        __syncthreads();                                      // (the other buffer is written next: its readers are past this)
        y = buf[turn][tid ^ J];
        turn ^= 1;
    } else {
        y = (uint64_t)from_lane_xor<J>((uint32_t)(x >> 32)) << 32 | from_lane_xor<J>((uint32_t)x);
    }
    const bool keep_min = ((tid & K) == 0) == ((tid & J) == 0);
    x = (x < y) == keep_min ? x : y;                          // (keys are distinct: they end in the index)
    if constexpr (J > 1) sort_step<K, J / 2>(x, tid, buf, turn);
}
template <int K>
__device__ __forceinline__ void sort_merge(uint64_t &x, int tid, uint64_t (*buf)[CS_LEN], int &turn)
{
    if constexpr (K > 2) sort_merge<K / 2>(x, tid, buf, turn);
    sort_step<K, K / 2>(x, tid, buf, turn);
}

// Array a of the launch: a < n_mats -> the rows of matrix a, else the columns of matrix a - n_mats.  Chunks of a piece in
// ascending (key, index) order to keys / idx (indexed as the scores; idx counts from the piece's start); a piece of one
// chunk is finished here.
__global__ __launch_bounds__(CS_THREADS)
void chunk_sort_kernel(SortArrays s, const float *__restrict__ scores, uint32_t *__restrict__ keys, uint32_t *__restrict__ idx)
{
    __shared__ uint64_t buf[2][CS_LEN];
    const int tid = threadIdx.x;
    const SortArray ar = sort_array(s, (int)blockIdx.x / s.per);
    const int first = (int)blockIdx.x % s.per;
    if (ar.mode == ARR_SKIP) return;
    if (ar.mode == ARR_IDENTITY) {
        for (int i = first * CS_THREADS + tid; i < ar.n; i += s.per * CS_THREADS) ar.perm[i] = i;
        return;
    }
    const int cpp = (ar.piece + CS_LEN - 1) / CS_LEN, total = (ar.n + ar.piece - 1) / ar.piece * cpp;
    int turn = 0;
    for (int t = first; t < total; t += s.per) {              // (uniform over the workgroup)
        const int p0 = t / cpp * ar.piece, c0 = t % cpp * CS_LEN;
        const int len = min(CS_LEN, min(ar.piece, ar.n - p0) - c0), at = p0 + c0;
        // what fills up the chunk goes behind every channel
        const uint32_t k = tid < len ? sort_key(scores[ar.off + at + tid]) : ~0u;
        uint64_t x = (uint64_t)k << 32 | (uint32_t)tid;
        sort_merge<CS_LEN>(x, tid, buf, turn);
        if (tid < len) {
            if (cpp == 1) {
                ar.perm[at + tid] = at + (int)(uint32_t)x;
            } else {
                keys[ar.off + at + tid] = (uint32_t)(x >> 32);
                idx[ar.off + at + tid] = (uint32_t)c0 + (uint32_t)x;
            }
        }
    }
}

// Pieces of several sorted chunks: every channel's rank, and the permutation.
__global__ __launch_bounds__(RK_THREADS)
void rank_kernel(SortArrays s, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ idx)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t piece_keys[];    // all chunks of the piece
    const int tid = threadIdx.x;
    const SortArray ar = sort_array(s, (int)blockIdx.x / s.per);
    const int cpp = (ar.piece + CS_LEN - 1) / CS_LEN;
    if (ar.mode != ARR_SORT || cpp == 1) return;
    const int halves = (ar.piece + RK_THREADS - 1) / RK_THREADS, total = (ar.n + ar.piece - 1) / ar.piece * halves;
    int have = -1;
    for (int t = (int)blockIdx.x % s.per; t < total; t += s.per) {
        const int p0 = t / halves * ar.piece, e0 = t % halves * RK_THREADS, len = min(ar.piece, ar.n - p0);
        if (p0 != have) {                                     // (uniform over the workgroup)
            __syncthreads();                                  // the piece before has been read
            for (int i = tid; i < cpp * CS_LEN; i += RK_THREADS) piece_keys[i] = i < len ? keys[ar.off + p0 + i] : ~0u;
            __syncthreads();
            have = p0;
        }
        const int e = e0 + tid, own = e0 / CS_LEN;
        const uint32_t k = piece_keys[e];                     // (e < cpp * CS_LEN)
        int rank = e & (CS_LEN - 1);
        // keys of a chunk that go before k: those below it and, in the chunks before (lower indices), those equal to it
        auto count = [&](const uint32_t *c, auto before) {
            int b = 0;
#pragma unroll
            for (int w = CS_LEN / 2; w >= 1; w >>= 1) b += before(c[b + w - 1]) ? w : 0;
            return b + (before(c[b]) ? 1 : 0);
        };
#pragma unroll 4
        for (int c = 0; c < own; ++c) rank += count(piece_keys + c * CS_LEN, [&](uint32_t v) { return v <= k; });
#pragma unroll 4
        for (int c = own + 1; c < cpp; ++c) rank += count(piece_keys + c * CS_LEN, [&](uint32_t v) { return v < k; });
        if (e < len) ar.perm[p0 + rank] = p0 + (int)idx[ar.off + p0 + e];
    }
}

// ---- coupled reordering (paper App. "Channel Reordering": one permutation for all the matrix
// dimensions that carry the same activation; the scores of the coupled dimensions are summed) ----
// Arrays are numbered as in the sort kernel.  arr_next[a]: the next member of a's group, or -1.
// The leader (first member) of a group accumulates, member after member in array order:
//   s[leader][j] = (..(s[leader][j] + s[m1][j]) + s[m2][j]) + ...
// A member with repeat r > 1 is r times as long: each piece of seg channels of the group stands
// for r consecutive pieces of the member (one value head serving r query heads); its r scores of
// channel j are added one after the other, lower piece first.
__global__ __launch_bounds__(256)
void group_sum_kernel(const MatDesc *__restrict__ descs, int n_mats, int64_t sum_rows, float *__restrict__ scores,
                      const int *__restrict__ arr_mode, const int *__restrict__ arr_next,
                      const int *__restrict__ arr_seg, const int *__restrict__ arr_rep)
{
    const int a = blockIdx.y;
    if (arr_mode[a] != ARR_SORT || arr_next[a] < 0) return;      // only leaders with other members
    const bool is_row = a < n_mats;
    const MatDesc &d = descs[is_row ? a : a - n_mats];
    const int n = (int)(is_row ? d.rows : d.cols);
    const int sg = arr_seg[a];
    const int64_t off = is_row ? d.row_off : sum_rows + d.col_off;
    for (int j = (int)(blockIdx.x * blockDim.x + threadIdx.x); j < n; j += (int)(gridDim.x * blockDim.x)) {
        float acc = scores[off + j];
        for (int b = arr_next[a]; b >= 0; b = arr_next[b]) {
            const bool br = b < n_mats;
            const MatDesc &e = descs[br ? b : b - n_mats];
            const float *sb = scores + (br ? e.row_off : sum_rows + e.col_off);
            const int r = arr_rep[b];
            if (r == 1) {
                acc = acc + sb[j];
            } else {                                             // sg > 0 (checked on the host)
                const int64_t base = (int64_t)(j / sg) * r * sg + j % sg;
                for (int t = 0; t < r; ++t) acc = acc + sb[base + (int64_t)t * sg];
            }
        }
        scores[off + j] = acc;
    }
}

// the members of a group take their leader's permutation; a member with repeat r applies the
// permutation of group piece p inside each of its pieces r*p .. r*p + r - 1
__global__ __launch_bounds__(256)
void replicate_perm_kernel(const MatDesc *__restrict__ descs, int n_mats, int32_t *__restrict__ row_perm,
                           int32_t *__restrict__ col_perm, const int *__restrict__ arr_mode,
                           const int *__restrict__ arr_leader, const int *__restrict__ arr_seg,
                           const int *__restrict__ arr_rep)
{
    const int a = blockIdx.y;
    if (arr_mode[a] != ARR_SKIP) return;
    const int l = arr_leader[a];
    const bool ar = a < n_mats, lr = l < n_mats;
    const MatDesc &d = descs[ar ? a : a - n_mats];
    const MatDesc &e = descs[lr ? l : l - n_mats];
    const int n = (int)(ar ? d.rows : d.cols);
    const int r = arr_rep[a], sg = arr_seg[l];
    int32_t *dst = ar ? row_perm + d.row_off : col_perm + d.col_off;
    const int32_t *src = lr ? row_perm + e.row_off : col_perm + e.col_off;
    for (int j = (int)(blockIdx.x * blockDim.x + threadIdx.x); j < n; j += (int)(gridDim.x * blockDim.x)) {
        if (r == 1) {
            dst[j] = src[j];
        } else {
            const int pc = j / sg, dd = j - pc * sg;             // the member's piece and the channel inside it
            const int gbase = (pc / r) * sg;                     // first channel of the group's piece
            dst[j] = pc * sg + (src[gbase + dd] - gbase);
        }
    }
}

// ================================================================ gather
constexpr int GA_LDS_TARGET = 48 * 1024;            // rows per workgroup are chosen to fill about this much

// T = uint16_t (bf16) or float.  A workgroup stages rpw consecutive output rows of one matrix
// (their source rows) in LDS and emits them permuted; the column indices are read once per
// column chunk and serve all rpw rows.  A launch covers the matrices of one "class" (equal
// column count, hence equal LDS need): members[] lists them, wg_start[] is their workgroup prefix.
// Bound by HBM: the rows come in by direct loads to LDS, all of a workgroup's rows under way at once (through registers a
// wave had one load of 1 KiB in flight), and the column indices of a thread are requested a chunk ahead, the first behind
// the rows.  Through registers -> now: 8192 x 28672 fp32 477 -> 341 us (5.5 TB/s), bf16 197 -> 171; 8192 x 14336 193 -> 163
// and 98 -> 88; 16384 x 2048 57 -> 47 and 40 -> 25.
template <class T, int TH>
__global__ __launch_bounds__(TH)
void gather_kernel(const MatDesc *__restrict__ descs, MatDesc one, const int *__restrict__ members,
                   const int *__restrict__ wg_start, int n_members, int rpw,
                   const int32_t *__restrict__ row_perm, const int32_t *__restrict__ col_perm,
                   T *__restrict__ out_all)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int V = 16 / sizeof(T);               // elements per 128-bit access
    typedef const T __attribute__((address_space(1))) *gtp;

    int mem = 0;
    if (descs) mem = find_matrix(wg_start, n_members, (int)blockIdx.x);
    const MatDesc &d = descs ? descs[members[mem]] : one;
    const int R = (int)d.rows, C = (int)d.cols;
    const int i0 = ((int)blockIdx.x - (descs ? wg_start[mem] : 0)) * rpw;     // first output row
    const int nr = min(rpw, R - i0);
    const T *in = sizeof(T) == 2 ? reinterpret_cast<const T *>(d.w) : reinterpret_cast<const T *>(d.s);
    const int64_t ld = sizeof(T) == 2 ? d.ld_w : d.ld_s;
    const int32_t *__restrict__ rp = row_perm + d.row_off;
    const int32_t *__restrict__ cp = col_perm + d.col_off;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int bytes = C * (int)sizeof(T), pieces = (bytes + 1023) / 1024;       // a row takes whole KiB of LDS
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    // Source rows: one load, a row per lane (at most 8).  An index loaded per piece is a wait per piece, and with one long row
    // per workgroup that chain is longer than the row's own loads (8192 x 28672: bf16 202 us, fp32 369).  A permutation
    // never trips the clamp; it keeps a bad one in bounds.
    const int source = min(max(rp[i0 + min(lane, nr - 1)], 0), R - 1);
    int r = wave / pieces, p = wave - r * pieces;             // this wave's piece: 1 KiB of a row, one per turn
    while (r < nr) {
        const T *src = in + (int64_t)__builtin_amdgcn_readlane(source, r) * ld;
        const uint32_t at = (uint32_t)(r * pieces + p) * 1024u;
        if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {   // (lanes past the row's end: its last 16 bytes, into the padding)
            const uint32_t off = min((uint32_t)p * 1024u + (uint32_t)lane * 16u, (uint32_t)bytes - 16u);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(reinterpret_cast<const char *>(src) + off),
                                             (__attribute__((address_space(3))) void *)(lds0 + at), 16, 0, 2);
        } else {
            for (int j = lane; j < 1024 / (int)sizeof(T); j += 64) {
                const int c = p * (1024 / (int)sizeof(T)) + j;
                if (c < C) reinterpret_cast<T *>(smem + at)[j] = *(gtp)(src + c);
            }
        }
        for (p += TH / 64; p >= pieces; p -= pieces) ++r;
    }
    struct Index { int4 a, b; };
    auto indices = [&](int j) {
        Index o;
        j = min(j, C - V);
        o.a = *reinterpret_cast<const int4 *>(cp + j);
        if constexpr (V == 8) o.b = *reinterpret_cast<const int4 *>(cp + j + 4);
        return o;
    };
    const int j0 = (int)threadIdx.x * V;
    Index next = indices(j0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this wave's pieces (and its first indices)
    __syncthreads();
    T *dst = out_all + d.elem_off + (int64_t)i0 * C;      // dense output, C % 8 == 0: 16-byte aligned rows
    for (int j = j0; j < C; j += TH * V) {
        const Index ix = next;
        next = indices(j + TH * V);
        int ci[V];
        ci[0] = ix.a.x; ci[1] = ix.a.y; ci[2] = ix.a.z; ci[3] = ix.a.w;
        if constexpr (V == 8) { ci[4] = ix.b.x; ci[5] = ix.b.y; ci[6] = ix.b.z; ci[7] = ix.b.w; }
        for (int r = 0; r < nr; ++r) {
            const T *srcl = reinterpret_cast<const T *>(smem + (size_t)r * pieces * 1024);
            T tmp[V];
#pragma unroll
            for (int e = 0; e < V; ++e) tmp[e] = srcl[ci[e]];
            // written once, not read again by this kernel: streamed past the caches
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4_t *>(tmp),
                                        (__attribute__((address_space(1))) u32x4_t *)(dst + (int64_t)r * C + j));
        }
    }
}

static int gather_rows_per_wg(int64_t C, size_t elem)
{
    int64_t r = GA_LDS_TARGET / (C * (int64_t)elem);
    return (int)(r < 1 ? 1 : (r > 8 ? 8 : r));
}

}  // namespace sbits

using namespace sbits;

// ---- workspace of the reorder stage (after the head) ---------------------------------
//   scores [L] | rowpart [RP] | colpart [CP] | keys [L] | idx [L]
// with L = channels (rows + cols), RP = sum rows*npanel, CP = sum nband*cols.
struct ReorderWs {
    float *scores, *rowpart, *colpart;
    uint32_t *keys, *idx;
};

static size_t reorder_ws_layout(void *base, int64_t L, int64_t RP, int64_t CP, ReorderWs *out)
{
    char *p = static_cast<char *>(base);
    size_t b = 0;
    auto take = [&](size_t bytes) { char *q = p ? p + b : nullptr; b += sbits_align_up(bytes, 256); return q; };
    float *scores = reinterpret_cast<float *>(take((size_t)L * 4));
    float *rowpart = reinterpret_cast<float *>(take((size_t)RP * 4));
    float *colpart = reinterpret_cast<float *>(take((size_t)CP * 4));
    uint32_t *keys = reinterpret_cast<uint32_t *>(take((size_t)L * 4));
    uint32_t *idx = reinterpret_cast<uint32_t *>(take((size_t)L * 4));
    if (out) { out->scores = scores; out->rowpart = rowpart; out->colpart = colpart; out->keys = keys; out->idx = idx; }
    return b;
}

// workgroups of score_partial_kernel for a matrix with npanel panels and nband bands
int sbits_score_wgs(int npanel, int nband) { return nband * npanel; }

void sbits_score_geometry(int64_t R, int64_t C, int band_rows, int *npanel, int *nband)
{
    *npanel = (int)((C + SC_PANEL * SC_COLS - 1) / (SC_PANEL * SC_COLS));
    *nband = (int)((R + band_rows - 1) / band_rows);
}

// Rows per band for a plan of these matrices: 512, which leave the fewest partial sums, where they take no more turns of two workgroups a CU
// than bands of 256 (432 workgroups instead of 864: 527 us and 559; 104 instead of 208, half of the CUs idle: 180 and 130; 5 % is what the
// fewer sums are worth); else 256, halved while the workgroups, whose rows come one after the other, still find a CU each, or, where
// narrow matrices leave many of them with little to do, while their work fills 200 whole panels at most (and there were fewer than 192); and
// as long as one tree of 128 adds up a column.  Scores and permutations: 512 x 512 136 us with 256 rows, 34 with 8; 2048 x 2048 145 -> 47 (16 rows); 4096 x 4096
// 159 -> 58 (32); 2048 x 8192 twice 161 -> 60 (32).  The line: 128 workgroups take 123 us, halved 113; 144 take 130 and 147, 160 take
// 136 and 155 (in 288 and 320, a few CUs have two and the others wait); 166 with the work of 100 take 125, halved 119.  Over 550 drawn plans
// 3 % behind the best height; with 192 alone for the line, whatever their work, 4 %.
int sbits_score_rows(const int64_t *rows, const int64_t *cols, int n_mats)
{
    int64_t max_rows = 0, elems = 0;
    for (int i = 0; i < n_mats; ++i) {
        elems += rows[i] * cols[i];
        if (rows[i] > max_rows) max_rows = rows[i];
    }
    auto wgs = [&](int band) {
        int64_t w = 0;
        for (int i = 0; i < n_mats; ++i) {
            int npanel, nband;
            sbits_score_geometry(rows[i], cols[i], band, &npanel, &nband);
            w += sbits_score_wgs(npanel, nband);
        }
        return w;
    };
    const int64_t tall = wgs(SC_ROWS), half = wgs(SC_ROWS / 2);
    if (tall >= 400 && 95 * ((tall + 511) / 512) * 2 <= 100 * ((half + 511) / 512)) return SC_ROWS;
    int r = SC_ROWS / 2;
    auto halves = [&]() {
        const int64_t w = wgs(r / 2);
        return w <= 256 || (w <= 512 && half * (256 / r) < 192 && elems <= (int64_t)200 * (r / 2) * (SC_PANEL * SC_COLS));
    };
    while (r > 8 && max_rows <= 128 * (r / 2) && halves()) r >>= 1;
    return r;
}

size_t sbits_reorder_ws_bytes(int64_t L, int64_t RP, int64_t CP)
{
    return reorder_ws_layout(nullptr, L, RP, CP, nullptr);
}

// descriptor of a single matrix with its own (offset-free) layout
static MatDesc single_desc(const void *W, const float *S, int64_t R, int64_t C, int64_t ld_w, int64_t ld_s, int band_rows)
{
    MatDesc d;
    memset(&d, 0, sizeof d);
    d.w = static_cast<const uint16_t *>(W);
    d.s = S;
    d.rows = R; d.cols = C; d.ld_w = ld_w; d.ld_s = ld_s;
    sbits_score_geometry(R, C, band_rows, &d.npanel, &d.nband);
    return d;
}

static int run_scores(sbits_ctx *ctx, const MatDesc *descs, const MatDesc &one, const int *d_wg_start,
                      int n_mats, int total_wg, int band_rows, int64_t sum_rows, int64_t sum_cols, const ReorderWs &w)
{
    auto launch = [&](auto *kernel, int ring) -> int {
        const size_t lds = (size_t)SC_THREADS / 64 * ring * 2 * SC_COLS * 4 + (size_t)band_rows * SC_PANEL * 4;
        if (lds > 65536) SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kernel, dim3((unsigned)total_wg), dim3(SC_THREADS), lds, ctx->stream, descs, one, d_wg_start, n_mats, band_rows,
                           w.rowpart, w.colpart);
        return SBITS_OK;
    };
    const int rc = band_rows == 512 ? launch(&score_partial_kernel<3>, 3)
                 : band_rows == 256 || total_wg > sbits_cus(ctx) ? launch(&score_partial_kernel<4>, 4) : launch(&score_partial_kernel<8>, 8);
    if (rc) return rc;
    SBITS_HIP(ctx, hipGetLastError());
    const int64_t L = sum_rows + sum_cols;
    hipLaunchKernelGGL(score_finish_kernel, dim3((unsigned)((L + 255) / 256)), dim3(256), 0, ctx->stream,
                       descs, one, n_mats, sum_rows, sum_cols, w.rowpart, w.colpart, w.scores,
                       w.scores + sum_rows);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

// max_len, max_piece: the longest array and the longest run of channels that is sorted as one
static int run_argsort(sbits_ctx *ctx, SortArrays s, int64_t max_len, int64_t max_piece, const ReorderWs &w)
{
    // A workgroup per (half) chunk of the longest array, up to a few thousand in all: with many arrays, most of them
    // shorter, the workgroups without work would take longer than the others (448 arrays of 1024 to 14336 channels: 221 us
    // with one per chunk of the longest, 162 us so).
    const int64_t na = 2 * (int64_t)s.n_mats;
    auto per = [&](int64_t len, int64_t most) {
        const int64_t c = (max_len + len - 1) / len, p = (most + na - 1) / na;
        return (int)(c < p ? c : p);
    };
    s.per = per(CS_LEN, 2048);
    hipLaunchKernelGGL(chunk_sort_kernel, dim3((unsigned)(na * s.per)), dim3(CS_THREADS), 0, ctx->stream, s, w.scores, w.keys, w.idx);
    SBITS_HIP(ctx, hipGetLastError());
    if (max_piece <= CS_LEN) return SBITS_OK;
    s.per = per(RK_THREADS, 4096);
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(&rank_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    hipLaunchKernelGGL(rank_kernel, dim3((unsigned)(na * s.per)), dim3(RK_THREADS), sbits_align_up((size_t)max_piece, CS_LEN) * 4,
                       ctx->stream, s, w.keys, w.idx);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

// ---- single matrix ----------------------------------------------------------------------
int sbits_launch_scores(sbits_ctx *ctx, const float *S, int64_t R, int64_t C, int64_t ld, int band_rows,
                        float *row_score, float *col_score, void *scratch)
{
    MatDesc one = single_desc(nullptr, S, R, C, C, ld, band_rows);
    ReorderWs w;
    reorder_ws_layout(scratch, R + C, R * one.npanel, (int64_t)one.nband * C, &w);
    int rc = run_scores(ctx, nullptr, one, nullptr, 1, sbits_score_wgs(one.npanel, one.nband), band_rows, R, C, w);
    if (rc) return rc;
    if (row_score)
        SBITS_HIP(ctx, hipMemcpyAsync(row_score, w.scores, (size_t)R * 4, hipMemcpyDeviceToDevice, ctx->stream));
    if (col_score)
        SBITS_HIP(ctx, hipMemcpyAsync(col_score, w.scores + R, (size_t)C * 4, hipMemcpyDeviceToDevice, ctx->stream));
    return SBITS_OK;
}

int sbits_launch_reorder(sbits_ctx *ctx, const float *S, int64_t R, int64_t C, int64_t ld, int band_rows,
                         int32_t *row_perm, int32_t *col_perm, void *scratch)
{
    MatDesc one = single_desc(nullptr, S, R, C, C, ld, band_rows);
    ReorderWs w;
    reorder_ws_layout(scratch, R + C, R * one.npanel, (int64_t)one.nband * C, &w);
    int rc = run_scores(ctx, nullptr, one, nullptr, 1, sbits_score_wgs(one.npanel, one.nband), band_rows, R, C, w);
    if (rc) return rc;
    const int64_t len = R > C ? R : C;
    return run_argsort(ctx, SortArrays{nullptr, one, 1, 1, R, nullptr, nullptr, row_perm, col_perm}, len, len, w);
}

// Workgroups of 512 threads, of 1024 where fewer than three fit a CU's LDS (fp32 8192 x 16384, two: 192 us against 198; 8192 x
// 32768, one: 380 against 391; bf16 8192 x 28672, two: no difference beyond the noise).
template <class T>
static int launch_gather(sbits_ctx *ctx, const MatDesc *descs, const MatDesc &one, const int *members, const int *wg_start,
                         int n_members, int64_t total_wg, int rpw, int64_t C, const int32_t *rp, const int32_t *cp, T *out)
{
    const size_t lds = (size_t)rpw * (((size_t)C * sizeof(T) + 1023) / 1024 * 1024);
    const bool large = lds > 53 * 1024;
    auto *fn = large ? &gather_kernel<T, 1024> : &gather_kernel<T, 512>;
    SBITS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    hipLaunchKernelGGL(fn, dim3((unsigned)total_wg), dim3(large ? 1024 : 512), lds, ctx->stream, descs, one, members, wg_start,
                       n_members, rpw, rp, cp, out);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

int sbits_launch_gather(sbits_ctx *ctx, const void *W, const float *S, int64_t R, int64_t C,
                        int64_t ld_w, int64_t ld_s, const int32_t *rp, const int32_t *cp,
                        void *w_out, float *s_out)
{
    if ((size_t)C * 4 > 160 * 1024) return SBITS_ERR_BAD_SHAPE;
    MatDesc one = single_desc(W, S, R, C, ld_w, ld_s, SC_ROWS);
    int rc = SBITS_OK;
    if (w_out) {
        const int rpw = gather_rows_per_wg(C, 2);
        rc = launch_gather(ctx, nullptr, one, nullptr, nullptr, 1, (R + rpw - 1) / rpw, rpw, C, rp, cp, static_cast<uint16_t *>(w_out));
    }
    if (!rc && s_out) {
        const int rpw = gather_rows_per_wg(C, 4);
        rc = launch_gather(ctx, nullptr, one, nullptr, nullptr, 1, (R + rpw - 1) / rpw, rpw, C, rp, cp, s_out);
    }
    return rc;
}

// ---- all matrices of the plan (descriptor table already in the workspace head) ------------
int sbits_launch_reorder_all(sbits_plan *plan, int32_t *row_perm, int32_t *col_perm, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    ReorderWs w;
    reorder_ws_layout(sbits_scratch(plan, ws), plan->sum_rows + plan->sum_cols, plan->sum_rowpart,
                      plan->sum_colpart, &w);
    const int *d_pre = sbits_prefix_ptr(plan, ws, SLOT_SCORE_WGS);
    MatDesc none;
    memset(&none, 0, sizeof none);
    int rc = run_scores(ctx, sbits_desc_ptr(ws), none, d_pre, plan->n_mats, plan->score_wg_start.back(),
                        plan->score_rows, plan->sum_rows, plan->sum_cols, w);
    if (rc) return rc;
    const int64_t len = plan->max_rows > plan->max_cols ? plan->max_rows : plan->max_cols;
    return run_argsort(ctx, SortArrays{sbits_desc_ptr(ws), none, plan->n_mats, 1, plan->sum_rows, nullptr, nullptr, row_perm, col_perm},
                       len, len, w);
}

// Host part of the coupled reordering: validates the groups and builds, per array a (rows of matrix
// a, or columns of matrix a - n_mats), what the sort kernel does with it (mode), the piece length
// (seg), the next member of its group (next) and, for non-leaders, the group's first member (leader).
int sbits_coupling_tables(const sbits_plan *plan, const int32_t *row_group, const int32_t *col_group, int n_groups,
                          const int32_t *group_segment, const int32_t *row_repeat, const int32_t *col_repeat,
                          sbits_coupling *out)
{
    const int nm = plan->n_mats, na = 2 * nm;
    std::vector<int> mode(na), seg(na, 0), next(na, -1), leader(na, -1), rep(na, 1);
    std::vector<int> last(n_groups > 0 ? n_groups : 0, -1);
    std::vector<int> first(last);
    auto len = [&](int a) { return a < nm ? plan->rows[a] : plan->cols[a - nm]; };
    for (int a = 0; a < na; ++a) {
        const int g = a < nm ? row_group[a] : col_group[a - nm];
        const int32_t *rp = a < nm ? row_repeat : col_repeat;
        const int r = rp ? rp[a < nm ? a : a - nm] : 1;
        if (r < 1) return SBITS_ERR_INVALID_ARG;
        if (g == SBITS_DIM_INDEPENDENT || g == SBITS_DIM_FIXED) {
            if (r != 1) return SBITS_ERR_INVALID_ARG;
            mode[a] = g == SBITS_DIM_FIXED ? ARR_IDENTITY : ARR_SORT;
            continue;
        }
        if (g < 0 || g >= n_groups) return SBITS_ERR_INVALID_ARG;
        const int sg = group_segment ? group_segment[g] : 0;
        if (sg < 0) return SBITS_ERR_BAD_SHAPE;
        rep[a] = r;
        if (first[g] < 0) {
            if (r != 1) return SBITS_ERR_INVALID_ARG;              // the first member carries the group's length
            if (sg > 0 && len(a) % sg) return SBITS_ERR_BAD_SHAPE;
            first[g] = last[g] = a;
            mode[a] = ARR_SORT;
            seg[a] = sg;
        } else {
            if (r > 1 && sg == 0) return SBITS_ERR_BAD_SHAPE;     // repeats are repeats of pieces
            if (len(a) != (int64_t)r * len(first[g])) return SBITS_ERR_BAD_SHAPE;   // the same activation
            mode[a] = ARR_SKIP;
            leader[a] = first[g];
            next[last[g]] = a;
            last[g] = a;
        }
    }
    *out = sbits_coupling{mode, seg, next, leader, rep};
    return SBITS_OK;
}

// Coupled reordering of all matrices.  group[a] for every array a (rows of matrix a, or columns of
// matrix a - n_mats): SBITS_DIM_INDEPENDENT, SBITS_DIM_FIXED or a group id; segment[g]: 0 or the
// piece length for group g; repeat: pieces of the member per piece of the group.  The tables made of
// them are in the workspace head.
int sbits_launch_reorder_coupled_all(sbits_plan *plan, const sbits_coupling &cpl, int32_t *row_perm, int32_t *col_perm, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    const int nm = plan->n_mats, na = 2 * nm;
    const int *d_mode = sbits_prefix_ptr(plan, ws, SLOT_ARR_MODE), *d_seg = sbits_prefix_ptr(plan, ws, SLOT_ARR_SEG);
    const int *d_next = sbits_prefix_ptr(plan, ws, SLOT_ARR_NEXT), *d_leader = sbits_prefix_ptr(plan, ws, SLOT_ARR_LEADER);
    const int *d_rep = sbits_prefix_ptr(plan, ws, SLOT_ARR_REP);
    ReorderWs w;
    reorder_ws_layout(sbits_scratch(plan, ws), plan->sum_rows + plan->sum_cols, plan->sum_rowpart,
                      plan->sum_colpart, &w);
    const int *d_pre = sbits_prefix_ptr(plan, ws, SLOT_SCORE_WGS);
    MatDesc none;
    memset(&none, 0, sizeof none);
    const MatDesc *descs = sbits_desc_ptr(ws);
    int rc = run_scores(ctx, descs, none, d_pre, nm, plan->score_wg_start.back(), plan->score_rows, plan->sum_rows, plan->sum_cols, w);
    if (rc) return rc;
    const int64_t maxlen = plan->max_rows > plan->max_cols ? plan->max_rows : plan->max_cols;
    const dim3 g2((unsigned)((maxlen + 255) / 256), (unsigned)na);
    hipLaunchKernelGGL(group_sum_kernel, g2, dim3(256), 0, ctx->stream, descs, nm, plan->sum_rows, w.scores,
                       d_mode, d_next, d_seg, d_rep);
    int64_t max_piece = 1;
    for (int a = 0; a < na; ++a) {
        const int64_t len = cpl.mode[a] != ARR_SORT ? 1 : cpl.seg[a] > 0 ? cpl.seg[a] : a < nm ? plan->rows[a] : plan->cols[a - nm];
        if (len > max_piece) max_piece = len;
    }
    rc = run_argsort(ctx, SortArrays{descs, none, nm, 1, plan->sum_rows, d_mode, d_seg, row_perm, col_perm}, maxlen, max_piece, w);
    if (rc) return rc;
    hipLaunchKernelGGL(replicate_perm_kernel, g2, dim3(256), 0, ctx->stream, descs, nm, row_perm, col_perm,
                       d_mode, d_leader, d_seg, d_rep);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

// Matrices grouped by column count: members and workgroup prefixes of the weights' and the sensitivities' launches,
// class after class (each class has n_k + 1 prefix entries).
void sbits_gather_tables(sbits_plan *plan)
{
    std::vector<int64_t> classes;
    for (int i = 0; i < plan->n_mats; ++i) {
        bool seen = false;
        for (int64_t c : classes) seen = seen || c == plan->cols[i];
        if (!seen) classes.push_back(plan->cols[i]);
    }
    for (int64_t c : classes) {
        sbits_plan::GatherClass gc;
        gc.cols = c;
        gc.first = (int)plan->gather_members.size();
        gc.pre_first = (int)plan->gather_pre_w.size();
        gc.rpw_w = gather_rows_per_wg(c, 2);
        gc.rpw_s = gather_rows_per_wg(c, 4);
        int64_t tw = 0, ts = 0;
        gc.n = 0;
        for (int i = 0; i < plan->n_mats; ++i) {
            if (plan->cols[i] != c) continue;
            plan->gather_members.push_back(i);
            plan->gather_pre_w.push_back((int)tw);
            plan->gather_pre_s.push_back((int)ts);
            tw += (plan->rows[i] + gc.rpw_w - 1) / gc.rpw_w;
            ts += (plan->rows[i] + gc.rpw_s - 1) / gc.rpw_s;
            ++gc.n;
        }
        if (tw > 0x7fffffff || ts > 0x7fffffff) {
            plan->gather_members.clear(); plan->gather_pre_w.clear(); plan->gather_pre_s.clear(); plan->gather_classes.clear();
            return;
        }
        plan->gather_pre_w.push_back((int)tw);
        plan->gather_pre_s.push_back((int)ts);
        plan->gather_classes.push_back(gc);
    }
}

// One launch per class of matrices with equal column count (equal LDS need) and element type.
int sbits_launch_gather_all(sbits_plan *plan, const int32_t *row_perm, const int32_t *col_perm,
                            void *w_re, float *s_re, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    if ((size_t)plan->max_cols * 4 > 160 * 1024 || plan->gather_classes.empty()) return SBITS_ERR_BAD_SHAPE;
    const int *d_mem = sbits_prefix_ptr(plan, ws, SLOT_GATHER_MEMBERS);
    const int *d_pw = sbits_prefix_ptr(plan, ws, SLOT_GATHER_WGS_W), *d_ps = sbits_prefix_ptr(plan, ws, SLOT_GATHER_WGS_S);
    MatDesc none;
    memset(&none, 0, sizeof none);
    const MatDesc *descs = sbits_desc_ptr(ws);
    for (const sbits_plan::GatherClass &gc : plan->gather_classes) {
        int rc = SBITS_OK;
        if (w_re)
            rc = launch_gather(ctx, descs, none, d_mem + gc.first, d_pw + gc.pre_first, gc.n, plan->gather_pre_w[gc.pre_first + gc.n],
                               gc.rpw_w, gc.cols, row_perm, col_perm, static_cast<uint16_t *>(w_re));
        if (!rc && s_re)
            rc = launch_gather(ctx, descs, none, d_mem + gc.first, d_ps + gc.pre_first, gc.n, plan->gather_pre_s[gc.pre_first + gc.n],
                               gc.rpw_s, gc.cols, row_perm, col_perm, s_re);
        if (rc) return rc;
    }
    return SBITS_OK;
}
