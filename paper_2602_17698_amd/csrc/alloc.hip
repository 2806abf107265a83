// Scalable greedy bitwidth search (paper Algorithm 2, relaxed step Eq. 5) on the
// block x bitwidth cost table, run on the device by ONE launch.
//
// Per iteration:
//   keys    : marginal cost change per bit of raising / lowering every block,
//             read off the table at the current levels (Alg. 2 line 5), encoded
//             as 64-bit keys  [ordered value : 32][N-1-index : IB][step bits : 8]
//             so that "larger key" = "earlier in (value, lower index first)".
//             After the first iteration only the blocks that moved get new ones.
//   select  : the longest prefix of the descending key order that keeps
//             count <= cnt_max and cumulative step bits <= w_max.  Each round
//             splits the interval that holds the boundary into bins, sums counts
//             and step bits per bin and keeps the bin in which the prefix ends.
//   expansion (Alg. 2 lines 6-7)  : top-k raised, capped by the remaining
//             budget and by gain > 0.
//   swap (Alg. 2 lines 9-12)      : top-k/2 raised, bottom-k/2 (outside the
//             raised set) lowered; accepted iff the summed cost change, held in
//             order-independent int64 fixed point, is strictly negative; on
//             rejection k is halved.
// All sums that decide anything are integers, so results do not depend on the
// order in which atomics land.
//
// What bounds it: the chain of rounds (two to three per selection, one or two selections per
// iteration), not bytes.  With a launch per round an empty one cost 2 us and one with work 5 to 16 us
// (state re-read from memory, ticket, the last workgroup's serial scan), and an iteration took up to
// 20 of them and the host's answer.  Here G workgroups own a slice of the blocks each, in registers where it
// fits, and stay for the whole search; what they exchange (histograms, sums) goes through device-scope atomics
// into one of three rotating buffers, followed by a counter that all of them wait for, and every
// workgroup draws the same conclusions from the same sums.  No fence: nothing else is shared, so no cache has to be
// written back or invalidated.  A round takes 4 to 6 us that way, 2 us within one workgroup (512 threads: a
// wave's share of the scan is repeated per wave; 1024 threads spill and 256 leave the LDS atomics too few waves).
// Whole searches, launch per round before -> now: 107 k blocks, 24 iterations 2.72 -> 0.75 ms; 430 k blocks, 22 iterations
// 2.27 -> 0.79 ms; 4.2 M blocks 4.9 -> 3.6 ms; one proposal on 430 k blocks 157 -> 72 us.
#include <math.h>
#include <string.h>

#include "alloc_split.hpp"
#include "sbits_internal.hpp"

namespace sbits {

constexpr int AL_THREADS = 512;
constexpr int AL_WAVES = AL_THREADS / 64;
constexpr int64_t TRACE_CAP = 16384;
constexpr int SEL_DB = 10;                    // digit bits of a selection round
constexpr int SEL_BINS = 1 << SEL_DB;
constexpr int AL_KPT = 8;                     // blocks a thread holds in registers, or has in flight from memory
constexpr int AL_BPT = SEL_BINS / AL_THREADS;       // bins per thread
constexpr int AL_SUMS = 8;                    // values of one reduction

enum { MODE_NONE = 0, MODE_EXPAND = 1, MODE_ACCEPT = 2 };

struct AllocHead {
    long long N, T, k, kmin, used;
    int K, IB, l0, max_iters, done, mode;
    int ceil_log2_n;
    int bits[MAX_CAND];
    unsigned long long tauE, tauU, tauD, tauU2;   // the single step on caller-supplied estimates: what it raises and lowers
    unsigned int aborted;                     // workgroups that gave up waiting for the others: if any, nothing here is valid
    unsigned int pad_;
};
// What the host learns: written to page-locked host memory by the workgroup that leads, so that it takes neither a copy nor
// a wait of its own.
struct AllocResult {
    long long k, used, budget, cost_fixed, bits_check;
    long long prop_up, prop_dn, prop_after;
    int shift, status, iters, expansions, swaps_ok, swaps_rej, mode, valid;
};
// One exchange between the workgroups; three of them take turns (see grid_sync).
struct AllocXchg {
    unsigned long long hist[SEL_BINS];        // per bin: (sum of step widths << 32) | number of keys
    unsigned long long sum[AL_SUMS];
};
struct AllocState {
    AllocHead head;
    unsigned int arrived;                     // workgroups that reached the current exchange, counted on (past 32 bits: from 0 again)
    unsigned int pad_[63];
    AllocXchg x[3];
};

// What the count of arrivals starts from.
#ifndef SBITS_FIRST_ARRIVALS
#define SBITS_FIRST_ARRIVALS 0u
#endif

// The start state from a kernel argument: no host buffer has to outlive the call, so nothing waits.
__global__ __launch_bounds__(AL_THREADS)
void set_state_kernel(AllocState *st, AllocHead head)
{
    if (threadIdx.x == 0) { st->head = head; st->arrived = SBITS_FIRST_ARRIVALS; }
    unsigned long long *j = reinterpret_cast<unsigned long long *>(st->x);
    for (unsigned i = threadIdx.x; i < sizeof(st->x) / 8; i += AL_THREADS) j[i] = 0ull;
}

__device__ __forceinline__ unsigned int ord_f32(float f)
{
    const unsigned int u = __float_as_uint(f + 0.0f);          // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ long long fx(float v, int shift)
{
    const double p2 = __longlong_as_double((long long)(1023 + shift) << 52);
    return __double2ll_rn((double)v * p2);
}

typedef unsigned long long u64;

__device__ __forceinline__ u64 dev_load(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void dev_store(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// values that are the same in every lane, said so to the compiler (they would fill the vector registers)
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ u64 uni(u64 v) { return (u64)(unsigned)uni((int)(v >> 32)) << 32 | (unsigned)uni((int)v); }

// One workgroup's view of the search.  Everything but the slice and the keys is the same in all of them.
struct Team {
    AllocState *st;
    int G, g;                     // workgroups, this one
    long long n0, n1;             // its blocks
    unsigned int turn;            // exchanges so far
    int spin_limit;
    bool ok;                      // false: a wait was given up, leave
};

struct AllocShared {
    u64 hist[SEL_BINS];
    alignas(16) int wave_c[AL_WAVES], wave_w[AL_WAVES];
    u64 sum[AL_SUMS];
    int above_c, above_w, at_cnt, boundary;
    int ok;
    int bits[MAX_CAND];
};

__device__ __forceinline__ AllocXchg *xchg(const Team &t) { return &t.st->x[t.turn % 3u]; }

// All workgroups have added their part to the exchange buffer of this turn; afterwards its sums are
// complete for everybody.  The atomics are performed at the point of coherence: waiting for their
// acknowledgement (vmcnt) orders them before the arrival.
// The wait is bounded: if a workgroup gets no place on the device, the others leave, each after its own wait, at this
// exchange or the next one; so do those that start later, at their first exchange that somebody is missing from.
__device__ __forceinline__ void grid_sync(Team &t, AllocShared &sh)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int target = SBITS_FIRST_ARRIVALS + (unsigned int)t.G * (t.turn + 1u);
        (void)__hip_atomic_fetch_add(&t.st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned int seen;
        int left = t.spin_limit;
        // (the count is less than 2 G away from the target: the difference has a sign wherever 32 bits end)
        while ((int)((seen = __hip_atomic_load(&t.st->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) - target) < 0 && left-- > 0)
            __builtin_amdgcn_s_sleep(1);
        const bool ok = (int)(seen - target) >= 0;
        if (!ok) (void)__hip_atomic_fetch_add(&t.st->head.aborted, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.ok = ok;
    }
    __syncthreads();
    t.ok = uni(sh.ok) != 0;
}

// The end of a turn, after the sums were read.  The buffer of the turn before was read by everybody before
// they arrived at this one: it is cleared, and is in use again two turns later.
__device__ __forceinline__ void end_turn(Team &t)
{
    AllocXchg *old = &t.st->x[(t.turn + 2u) % 3u];
    const int per = (SEL_BINS + t.G - 1) / t.G;
    for (int b = t.g * per + (int)threadIdx.x; b < min((t.g + 1) * per, SEL_BINS); b += AL_THREADS) dev_store(&old->hist[b], 0ull);
    if (t.g == 0 && threadIdx.x < AL_SUMS) dev_store(&old->sum[threadIdx.x], 0ull);
    ++t.turn;
}

// Maxima of the first NMAX and sums of the other values over all threads of all workgroups; the same in every thread.
template <int NMAX, int NV>
__device__ __forceinline__ void team_reduce(Team &t, AllocShared &sh, u64 (&v)[NV])
{
    static_assert(NV <= AL_SUMS, "slots");
#pragma unroll
    for (int q = 0; q < NV; ++q)
        for (int off = 32; off; off >>= 1) {
            const u64 o = __shfl_xor(v[q], off);
            v[q] = q < NMAX ? (v[q] > o ? v[q] : o) : v[q] + o;
        }
    __syncthreads();
    if (threadIdx.x < NV) sh.sum[threadIdx.x] = 0ull;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            if (q < NMAX) atomicMax(&sh.sum[q], v[q]);
            else atomicAdd(&sh.sum[q], v[q]);
        }
    }
    __syncthreads();
    if (t.G > 1) {
        AllocXchg *x = xchg(t);
        if (threadIdx.x < NV) {
            const u64 o = sh.sum[threadIdx.x];
            if ((int)threadIdx.x < NMAX) atomicMax(&x->sum[threadIdx.x], o);
            else atomicAdd(&x->sum[threadIdx.x], o);
        }
        grid_sync(t, sh);
        if (threadIdx.x < NV) sh.sum[threadIdx.x] = dev_load(&x->sum[threadIdx.x]);
        end_turn(t);
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = uni(sh.sum[q]);
}

// the smallest s with span >> s < SEL_BINS
__device__ __forceinline__ int bin_shift(u64 span)
{
    const int len = 64 - __clzll((long long)(span | 1ull));
    return len > SEL_DB ? len - SEL_DB : 0;
}

struct Sel { u64 tau; int n_sel, w_sel; };           // selected <=> key >= tau

// A workgroup's blocks: their two keys (0: cannot be raised / lowered) and levels.  A thread owns blocks n0 + tid,
// n0 + tid + AL_THREADS, ... and nobody else touches what belongs to them.  RES: it holds all of them (at most
// AL_KPT) in registers; otherwise they live in memory and come in AL_KPT at a time.
struct Batch { u64 ku[AL_KPT], kd[AL_KPT]; int lv[AL_KPT]; };
template <bool RES>
struct Slice {
    Batch reg;                    // RES
    u64 *mu, *md;                 // [N] in the workspace
    uint8_t *level;
    long long n0, n1;

    // f(first block of the batch, batch): block u of it is first + u * AL_THREADS, there if < n1 (else its keys are 0).
    // What f changes is kept (WR) in all three arrays.  need_kd: f looks at keyD (from memory it is half of the bytes).
    template <bool LV, bool WR, class F>
    __device__ __forceinline__ void visit(F &&f, bool need_kd = true)
    {
        if constexpr (RES) {
            f(n0 + (int)threadIdx.x, reg);
        } else {
            for (long long i0 = n0 + (int)threadIdx.x; i0 < n1; i0 += (long long)AL_KPT * AL_THREADS) {
                Batch b;
#pragma unroll
                for (int u = 0; u < AL_KPT; ++u) {
                    const long long i = i0 + (long long)u * AL_THREADS;
                    b.ku[u] = i < n1 ? mu[i] : 0ull;
                    b.kd[u] = 0ull;
                    b.lv[u] = LV && i < n1 ? (int)level[i] : 0;
                }
                if (need_kd) {
#pragma unroll
                    for (int u = 0; u < AL_KPT; ++u) {
                        const long long i = i0 + (long long)u * AL_THREADS;
                        b.kd[u] = i < n1 ? md[i] : 0ull;
                    }
                }
                f(i0, b);
                if constexpr (WR) store(i0, b);
            }
        }
    }
    __device__ __forceinline__ void store(long long i0, const Batch &b)
    {
#pragma unroll
        for (int u = 0; u < AL_KPT; ++u) {
            const long long i = i0 + (long long)u * AL_THREADS;
            if (i < n1) { mu[i] = b.ku[u]; md[i] = b.kd[u]; level[i] = (uint8_t)b.lv[u]; }
        }
    }
    // the blocks for the first time
    template <class F>
    __device__ __forceinline__ void start(F &&f)
    {
        for (long long i0 = n0 + (int)threadIdx.x; i0 < n1; i0 += (long long)AL_KPT * AL_THREADS) {
            Batch b;
#pragma unroll
            for (int u = 0; u < AL_KPT; ++u) { b.ku[u] = b.kd[u] = 0ull; b.lv[u] = 0; }
            f(i0, b);
            if constexpr (RES) reg = b;
            else store(i0, b);
        }
    }
};

// inclusive prefix sum over the 64 lanes of a wave
__device__ __forceinline__ unsigned int wave_prefix(unsigned int v)
{
    auto add = [&](auto ctrl, auto rows) {
        v += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    };
    add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8
    add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1, 3
    add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2, 3
    return v;
}

// The longest prefix of the descending order of the blocks' keys >= key_min with at most cnt_max keys and at
// most w_max step bits: of the keyU, or (down) of the keyD of the blocks outside the set keyU >= excl_tau.
// v = key >> 8 is compared; the first round's bins cover [lo, hi), where nearly all values lie, and its
// outermost bins everything below and above, so values outside are found as well, a round later.
// Neither limit is negative.  sh.hist is all zero before and after.
template <bool RES>
__device__ __forceinline__ Sel select(Team &t, AllocShared &sh, Slice<RES> &own, bool down, u64 excl_tau, u64 key_min,
                                      int cnt_max, int w_max, u64 lo, u64 hi, int TB)
{
    const int tid = (int)threadIdx.x;
    Sel r;
    int c0 = 0, w0 = 0;                              // totals of the keys above the current interval
    u64 from = 0, to = 0;                            // the interval after the first round
    int sh_bin = 0;
    bool first = true;
    sh_bin = bin_shift(hi > lo ? hi - lo + 2 * ((hi - lo) >> (SEL_DB - 1)) : 0);   // (two bins are the outermost)
    for (;;) {
        own.template visit<false, false>([&](long long, const Batch &bt) {
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const u64 key = down ? bt.kd[q] : bt.ku[q];
                if (key < key_min) continue;                         // also drops what is past the end (key 0)
                if (down && bt.ku[q] >= excl_tau) continue;
                const u64 v = key >> 8;
                int bin;
                if (first) {
                    const u64 n = ((v - lo) >> sh_bin) + 1ull;
                    bin = v < lo ? 0 : (n < (u64)(SEL_BINS - 1) ? (int)n : SEL_BINS - 1);
                } else {
                    if (v < from || v >= to) continue;
                    bin = (int)((v - from) >> sh_bin);
                }
                atomicAdd(&sh.hist[SEL_BINS - 1 - bin], ((key & 255ull) << 32) | 1ull);   // descending: the top bin first
            }
        }, down);
        __syncthreads();
        if (t.G > 1) {
            AllocXchg *x = xchg(t);
#pragma unroll
            for (int q = 0; q < AL_BPT; ++q) {
                const u64 v = sh.hist[tid + q * AL_THREADS];
                if (v) (void)__hip_atomic_fetch_add(&x->hist[tid + q * AL_THREADS], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            grid_sync(t, sh);
            u64 v[AL_BPT];
#pragma unroll
            for (int q = 0; q < AL_BPT; ++q) v[q] = dev_load(&x->hist[tid + q * AL_THREADS]);
#pragma unroll
            for (int q = 0; q < AL_BPT; ++q) sh.hist[tid + q * AL_THREADS] = v[q];
            end_turn(t);
            if (!t.ok) { r.tau = ~0ull; r.n_sel = r.w_sel = 0; return r; }
            __syncthreads();
        }
        // Sums over the bins above each bin (at most 2^24 keys of width <= 8: neither can reach 2^31); a thread has
        // AL_BPT consecutive bins.
        int mc[AL_BPT], mw[AL_BPT], tc = 0, tw = 0;
#pragma unroll
        for (int q = 0; q < AL_BPT; ++q) {
            const u64 v = sh.hist[tid * AL_BPT + q];
            mc[q] = (int)v; mw[q] = (int)(v >> 32);
            tc += mc[q]; tw += mw[q];
        }
#pragma unroll
        for (int q = 0; q < AL_BPT; ++q) sh.hist[tid * AL_BPT + q] = 0ull;
        int pc = (int)wave_prefix((unsigned)tc), pw = (int)wave_prefix((unsigned)tw);
        if ((tid & 63) == 63) { sh.wave_c[tid >> 6] = pc; sh.wave_w[tid >> 6] = pw; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < AL_WAVES - 1; ++w) {
            const bool before = w < (tid >> 6);
            pc += before ? sh.wave_c[w] : 0;
            pw += before ? sh.wave_w[w] : 0;
        }
        // The sums only grow downwards, so the first bin that does not fit whole is the one that does not fit while
        // everything above it does; it ends the prefix.
        int ac = c0 + pc - tc, aw = w0 + pw - tw;
#pragma unroll
        for (int q = 0; q < AL_BPT; ++q) {
            const int ic = ac + mc[q], iw = aw + mw[q];
            const bool fits = ic <= cnt_max && iw <= w_max;
            if (mc[q] && !fits && ac <= cnt_max && aw <= w_max) {
                sh.boundary = SEL_BINS - 1 - (tid * AL_BPT + q); sh.above_c = ac; sh.above_w = aw; sh.at_cnt = mc[q];
            } else if (q == AL_BPT - 1 && tid == AL_THREADS - 1 && fits) {
                sh.boundary = -1; sh.above_c = ic; sh.above_w = iw; sh.at_cnt = 0;
            }
            ac = ic; aw = iw;
        }
        __syncthreads();
        const int b = uni(sh.boundary), at = uni(sh.at_cnt);
        c0 = uni(sh.above_c); w0 = uni(sh.above_w);
        if (b < 0) {                                 // every key of the interval fits
            const u64 edge = first ? 0ull : from << 8;
            r.tau = edge > key_min ? edge : key_min;
            break;
        }
        if (first) {
            if (b == 0) { from = 0; to = lo; }
            else if (b == SEL_BINS - 1) { from = lo + ((u64)(SEL_BINS - 2) << sh_bin); to = 1ull << TB; }
            else { from = lo + ((u64)(b - 1) << sh_bin); to = from + (1ull << sh_bin); }
            first = false;
        } else {
            from += (u64)b << sh_bin;
            const u64 end = from + (1ull << sh_bin);
            to = end < to ? end : to;
        }
        if (at == 1 || to - from <= 1) {             // one key that does not fit: the prefix ends above it
            r.tau = to >> 56 ? ~0ull : to << 8;
            break;
        }
        sh_bin = bin_shift(to - from - 1);
    }
    r.n_sel = c0; r.w_sel = w0;
    return r;
}

__device__ __forceinline__ void trace_write(sbits_trace *tr, int it, int kind, long long k, long long n_up, long long n_dn,
                                            long long p_up, long long p_dn, long long before, long long after, long long delta)
{
    if (it >= TRACE_CAP) return;
    sbits_trace &t = tr[it];
    t.kind = kind; t.pad_ = 0; t.k = k; t.n_up = n_up; t.n_dn = n_dn; t.p_up = p_up; t.p_dn = p_dn;
    t.bits_before = before; t.bits_after = after; t.delta_fixed = delta;
}

// keys of block i at level l, whose table entries there, a level below and a level above are cl, cm and cp
__device__ __forceinline__ void table_keys(float cm, float cl, float cp, int l, int K, const int *bits, long long N, int IB,
                                           long long i, u64 &ku, u64 &kd)
{
    const u64 low = (u64)(N - 1 - i) << 8;
    ku = kd = 0;
    if (l < K - 1) {
        const int step = bits[l + 1] - bits[l];
        ku = ((u64)ord_f32((cl - cp) / (float)step) << (IB + 8)) | low | (unsigned)step;
    }
    if (l > 0) {
        const int step = bits[l] - bits[l - 1];
        kd = ((u64)(~ord_f32((cm - cl) / (float)step)) << (IB + 8)) | low | (unsigned)step;
    }
}

struct Ranges { u64 loU, hiU, loD, hiD; int TB, IB; };

// The sets of one iteration of Algorithm 2.  e: the expansion (not tried without slack): the first k blocks by
// keyU with a value above zero that fit the slack.  If it is empty, the balanced swap: u = the first h by keyU,
// d = the first h by keyD outside u, u2 = the longest prefix of u whose step bits fit the slack plus the bits d
// frees.  (One loop around one copy of the selection: inlined four times it spills.)  STEP: the levels are the caller's and
// may be over budget; the search's own never are.
template <bool STEP, bool RES>
__device__ __forceinline__ void choose_sets(Team &t, AllocShared &sh, Slice<RES> &own, long long k, long long slack,
                                            const Ranges &rg, Sel &e, Sel &u, Sel &d, Sel &u2)
{
    enum { EXPAND, UP, DOWN, UP2 };
    const int INF = 0x7fffffff;
    auto clip = [](long long v) { return (int)(v < -1 ? -1 : v > INF ? INF : v); };
    const u64 key_pos = (u64)0x80000001u << (rg.IB + 8);             // value > +0
    const int kc = clip(k), h = k / 2 < 1 ? 1 : clip(k / 2);
    e = u = d = u2 = Sel{~0ull, 0, 0};
    int phase = slack > 0 ? EXPAND : UP;
    for (;;) {
        const bool down = phase == DOWN;
        const Sel r = select(t, sh, own, down, u.tau, phase == EXPAND ? key_pos : 1ull, phase == EXPAND ? kc : h,
                             phase == EXPAND ? clip(slack) : phase == UP2 ? clip(slack + d.w_sel) : INF, down ? rg.loD : rg.loU,
                             down ? rg.hiD : rg.hiU, rg.TB);
        if (!t.ok) return;
        if (phase == EXPAND) {
            e = r;
            if (e.n_sel > 0) return;
            phase = UP;
        } else if (phase == UP) {
            u = r;
            phase = DOWN;
        } else if (phase == DOWN) {
            d = r;
            u2 = u;
            if (u.w_sel <= slack + d.w_sel) return;                  // all of u fits
            if constexpr (STEP)
                if (slack + d.w_sel < 0) { u2 = Sel{~0ull, 0, 0}; return; }   // over by more than d frees: nothing of u does
            phase = UP2;
        } else {
            u2 = r;
            return;
        }
    }
}

// The range of the values above zero, from its largest (as an ordered 32-bit word) and the complement of its
// smallest: for the values themselves (keyU) and for their complements (keyD).  0 to 0 if there is none.
__device__ __forceinline__ void value_range(u64 omax, u64 omin_inv, int IB, u64 &loU, u64 &hiU, u64 &loD, u64 &hiD)
{
    const u64 omin = (u64)~(unsigned int)omin_inv;
    loU = omax ? omin << IB : 0; hiU = omax ? (omax + 1) << IB : 0;
    loD = omax ? (u64)~(unsigned int)omax << IB : 0; hiD = omax ? (omin_inv + 1) << IB : 0;
}

// The whole search (STEP = false), or one step of it on caller-supplied estimates s_up / s_down at level[]
// (STEP = true: the paper's own loop re-estimates them from a fresh gradient every iteration, Alg. 2 lines
// 4-5, and the acceptance test of lines 11-12 is the caller's, who owns the loss; level[] is only read).
// only_if_aborted: a second launch behind the first, with one workgroup, that does the work if the first
// one gave up.
template <bool STEP, bool RES>
__global__ __launch_bounds__(AL_THREADS)
void search_kernel(AllocState *st, const float *__restrict__ cost, const float *__restrict__ s_up,
                   const float *__restrict__ s_down, uint8_t *level, u64 *__restrict__ keyU, u64 *__restrict__ keyD,
                   sbits_trace *tr, AllocResult *result, int spin_limit, int only_if_aborted)
{
    __shared__ AllocShared sh;
    const int tid = (int)threadIdx.x;
    if (only_if_aborted && !st->head.aborted) return;
    Team t;
    t.st = st; t.G = (int)gridDim.x; t.g = (int)blockIdx.x; t.turn = 0; t.spin_limit = spin_limit; t.ok = true;
    const long long N = st->head.N, T = st->head.T;
    const int K = st->head.K, IB = st->head.IB;
    const long long per = (N + t.G - 1) / t.G;
    Slice<RES> own;
    own.mu = keyU; own.md = keyD; own.level = level;
    own.n0 = min(N, per * t.g);
    own.n1 = min(N, own.n0 + per);
    if constexpr (RES) {
#pragma unroll
        for (int u = 0; u < AL_KPT; ++u) { own.reg.ku[u] = own.reg.kd[u] = 0ull; own.reg.lv[u] = 0; }
    }
    for (int b = tid; b < SEL_BINS; b += AL_THREADS) sh.hist[b] = 0ull;
    if (tid < MAX_CAND) sh.bits[tid] = st->head.bits[tid];
    __syncthreads();
    const int *bits = sh.bits;
    const bool lead = blockIdx.x == 0 && tid == 0;
    long long used = st->head.used, k = st->head.k;
    Ranges rg;
    rg.TB = 32 + IB; rg.IB = IB;

    if constexpr (STEP) {
        u64 red[5] = {0, 0, 0, 0, 0};                // s_up: largest, smallest inverted; s_down: the same; bits in use
        // (The keys go to memory in either form: the kernel that applies the step reads them.  All loads of a batch are
        // requested before any is used, the estimates whether the level needs them or not: one level after the other, each
        // followed by its estimates, an expansion over 16.7 M blocks takes 100 us longer.)
        for (long long i0 = own.n0 + tid; i0 < own.n1; i0 += (long long)AL_KPT * AL_THREADS) {
            int lv[AL_KPT];
            float up[AL_KPT], dn[AL_KPT];
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const long long i = i0 + (long long)q * AL_THREADS;
                lv[q] = i < own.n1 ? (int)level[i] : 0;
                up[q] = i < own.n1 ? s_up[i] : 0.0f;
                dn[q] = i < own.n1 ? s_down[i] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const long long i = i0 + (long long)q * AL_THREADS;
                if (i >= own.n1) continue;
                const int l = min(lv[q], K - 1);
                red[4] += (u64)bits[l];
                const u64 low = (u64)(N - 1 - i) << 8;
                u64 ku = 0, kd = 0;
                if (l < K - 1) {
                    const unsigned int o = ord_f32(up[q]);
                    ku = ((u64)o << (IB + 8)) | low | (unsigned)(bits[l + 1] - bits[l]);
                    if (o > 0x80000000u) { red[0] = max(red[0], (u64)o); red[1] = max(red[1], (u64)~o); }
                }
                if (l > 0) {
                    const unsigned int o = ord_f32(dn[q]);
                    kd = ((u64)(~o) << (IB + 8)) | low | (unsigned)(bits[l] - bits[l - 1]);
                    if (o > 0x80000000u) { red[2] = max(red[2], (u64)o); red[3] = max(red[3], (u64)~o); }
                }
                keyU[i] = ku;
                keyD[i] = kd;
                if constexpr (RES) { own.reg.ku[q] = ku; own.reg.kd[q] = kd; }
            }
        }
        team_reduce<4>(t, sh, red);
        if (!t.ok) return;
        u64 q0, q1;
        value_range(red[0], red[1], IB, rg.loU, rg.hiU, q0, q1);
        value_range(red[2], red[3], IB, q0, q1, rg.loD, rg.hiD);
        used = (long long)red[4];
        Sel e, u, d, u2;
        choose_sets<STEP>(t, sh, own, k, T - used, rg, e, u, d, u2);
        if (!t.ok) return;
        // (a swap is a proposal: the caller accepts or rejects it)
        const int mode = e.n_sel > 0 ? MODE_EXPAND : u2.n_sel > 0 && d.n_sel > 0 ? MODE_ACCEPT : MODE_NONE;
        if (lead) {
            AllocHead &hd = st->head;
            hd.mode = mode;
            hd.tauE = e.tau; hd.tauU = u.tau; hd.tauD = d.tau; hd.tauU2 = u2.tau;
            if (result) {
                AllocResult r = {};
                r.used = used; r.budget = T;
                r.mode = mode;
                r.prop_up = mode == MODE_EXPAND ? e.n_sel : mode == MODE_ACCEPT ? u2.n_sel : 0;
                r.prop_dn = mode == MODE_ACCEPT ? d.n_sel : 0;
                r.prop_after = used + (mode == MODE_EXPAND ? e.w_sel : mode == MODE_ACCEPT ? u2.w_sel - d.w_sel : 0);
                r.valid = 1;
                *result = r;
            }
        }
    } else {
        const int l0 = st->head.l0;
        u64 red[3] = {0, 0, 0};                      // gains: largest, smallest inverted; the largest cost
        own.start([&](long long i0, Batch &bt) {
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const long long i = i0 + (long long)q * AL_THREADS;
                if (i >= own.n1) continue;
                const float *c = cost + i * K;
                float prev = 0.0f, cm = 0.0f, cl = 0.0f, cp = 0.0f;
                for (int l = 0; l < K; ++l) {
                    const float v = c[l];
                    if (v > 0.0f) red[2] = max(red[2], (u64)__float_as_uint(v));
                    if (l) {
                        const unsigned int o = ord_f32((prev - v) / (float)(bits[l] - bits[l - 1]));
                        if (o > 0x80000000u) { red[0] = max(red[0], (u64)o); red[1] = max(red[1], (u64)~o); }
                    }
                    if (l == l0 - 1) cm = v;
                    if (l == l0) cl = v;
                    if (l == l0 + 1) cp = v;
                    prev = v;
                }
                table_keys(cm, cl, cp, l0, K, bits, N, IB, i, bt.ku[q], bt.kd[q]);
                bt.lv[q] = l0;
            }
        });
        team_reduce<3>(t, sh, red);
        if (!t.ok) return;
        int shift = 0;
        if (red[2]) {
            const unsigned int b = (unsigned int)red[2];
            const int e = (int)(b >> 23);
            const int ilog = e ? e - 127 : (31 - __clz((int)(b & 0x7fffffu))) - 149;
            shift = 61 - st->head.ceil_log2_n - (ilog + 1);
        }
        value_range(red[0], red[1], IB, rg.loU, rg.hiU, rg.loD, rg.hiD);
        const long long kmin = st->head.kmin;
        const int max_iters = st->head.max_iters;
        int iters = 0, expansions = 0, swaps_ok = 0, swaps_rej = 0, status = SBITS_OK;
        bool done = st->head.done != 0;
        // The blocks that way(keyU, keyD) moves by +1 or -1 get their new level and keys.  (All loads of a batch are
        // requested before any is used.)
        auto move = [&](auto way) {
            own.template visit<true, true>([&](long long i0, Batch &bt) {
                int by[AL_KPT];
                float cm[AL_KPT], cl[AL_KPT], cp[AL_KPT];
#pragma unroll
                for (int q = 0; q < AL_KPT; ++q) {
                    const long long i = i0 + (long long)q * AL_THREADS;
                    by[q] = i < own.n1 ? way(bt.ku[q], bt.kd[q]) : 0;
                    cm[q] = cl[q] = cp[q] = 0.0f;
                    if (by[q]) {
                        const int l = bt.lv[q] + by[q];
                        const float *c = cost + i * K;
                        cl[q] = c[l];
                        cm[q] = c[max(l - 1, 0)];
                        cp[q] = c[min(l + 1, K - 1)];
                    }
                }
#pragma unroll
                for (int q = 0; q < AL_KPT; ++q)
                    if (by[q]) {
                        bt.lv[q] += by[q];
                        table_keys(cm[q], cl[q], cp[q], bt.lv[q], K, bits, N, IB, i0 + (long long)q * AL_THREADS, bt.ku[q], bt.kd[q]);
                    }
            });
        };
        while (!done) {
            Sel e, u, d, u2;
            choose_sets<STEP>(t, sh, own, k, T - used, rg, e, u, d, u2);
            if (!t.ok) return;
            if (e.n_sel > 0) {
                move([&](u64 ku, u64) { return ku >= e.tau ? 1 : 0; });
                if (lead) trace_write(tr, iters, 0, k, e.n_sel, 0, e.n_sel, 0, used, used + e.w_sel, 0);
                used += e.w_sel;
                ++expansions;
            } else {
                u64 lg[2] = {0, 0};                  // the swap's loss and gain
                auto way = [&](u64 ku, u64 kd) { return ku >= u2.tau ? 1 : (kd >= d.tau && !(ku >= u.tau)) ? -1 : 0; };
                own.template visit<true, false>([&](long long i0, const Batch &bt) {
                    int by[AL_KPT];
                    float hi[AL_KPT], lo[AL_KPT];    // the table entries below and above the step
#pragma unroll
                    for (int q = 0; q < AL_KPT; ++q) {
                        const long long i = i0 + (long long)q * AL_THREADS;
                        by[q] = i < own.n1 ? way(bt.ku[q], bt.kd[q]) : 0;
                        hi[q] = lo[q] = 0.0f;
                        if (by[q]) {
                            const float *c = cost + i * K + bt.lv[q] + (by[q] > 0 ? 0 : -1);
                            hi[q] = c[0];
                            lo[q] = c[1];
                        }
                    }
#pragma unroll
                    for (int q = 0; q < AL_KPT; ++q)
                        if (by[q]) lg[by[q] > 0] += (u64)fx(hi[q] - lo[q], shift);
                });
                team_reduce<0>(t, sh, lg);
                if (!t.ok) return;
                const long long delta = (long long)(lg[0] - lg[1]);
                if (u2.n_sel > 0 && d.n_sel > 0 && delta < 0) {
                    move(way);
                    if (lead)
                        trace_write(tr, iters, 1, k, u2.n_sel, d.n_sel, u2.n_sel, d.n_sel, used, used + u2.w_sel - d.w_sel, delta);
                    used += u2.w_sel - d.w_sel;
                    ++swaps_ok;
                } else {
                    if (lead) trace_write(tr, iters, 2, k, 0, 0, u2.n_sel, d.n_sel, used, used, delta);
                    k = k / 2;
                    ++swaps_rej;
                }
            }
            ++iters;
            if (k < kmin) done = true;
            else if (iters >= max_iters) { done = true; status = SBITS_ERR_MAX_ITERS; }
        }
        u64 fin[2] = {0, 0};                         // cost and bits of the final levels
        own.template visit<true, false>([&](long long i0, const Batch &bt) {
            float c[AL_KPT];
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const long long i = i0 + (long long)q * AL_THREADS;
                c[q] = 0.0f;
                if (i < own.n1) {
                    c[q] = cost[i * K + bt.lv[q]];
                    if constexpr (RES) level[i] = (uint8_t)bt.lv[q];
                }
            }
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q)
                if (i0 + (long long)q * AL_THREADS < own.n1) {
                    fin[0] += (u64)fx(c[q], shift);
                    fin[1] += (u64)bits[bt.lv[q]];
                }
        });
        team_reduce<0>(t, sh, fin);
        if (!t.ok) return;
        if (lead) {
            AllocResult r = {};
            r.used = used; r.k = k; r.budget = T; r.shift = shift; r.status = status;
            r.iters = iters; r.expansions = expansions; r.swaps_ok = swaps_ok; r.swaps_rej = swaps_rej;
            r.cost_fixed = (long long)fin[0]; r.bits_check = (long long)fin[1];
            r.valid = 1;
            *result = r;
        }
    }
}

// ---- the single step's result: the proposed levels -----------------------------------------
__global__ __launch_bounds__(256)
void step_apply_kernel(const AllocState *st, const u64 *__restrict__ keyU, const u64 *__restrict__ keyD,
                       const uint8_t *level_in, uint8_t *level_out)
{
    const AllocHead &hd = st->head;
    const int mode = hd.mode;
    const u64 tauE = hd.tauE, tauU = hd.tauU, tauD = hd.tauD, tauU2 = hd.tauU2;
    const long long N = hd.N;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
        const u64 ku = keyU[i], kd = keyD[i];
        int l = level_in[i];
        if (mode == MODE_EXPAND) {
            if (ku >= tauE) ++l;
        } else if (mode == MODE_ACCEPT) {
            if (ku >= tauU2) ++l;
            else if (kd >= tauD && !(ku >= tauU)) --l;
        }
        level_out[i] = (uint8_t)l;
    }
}

static int ceil_log2_ll(long long v) { int p = 0; while ((1ll << p) < v) ++p; return p; }

// A wait between workgroups polls this often before it is given up (about half a second).
#ifndef SBITS_SPIN_LIMIT
#define SBITS_SPIN_LIMIT (1 << 18)
#endif
// What a search that was given up is followed by: 1 the single workgroup's, 0 an error or no result (for tests).
#ifndef SBITS_SECOND_TRY
#define SBITS_SECOND_TRY 1
#endif

}  // namespace sbits

using namespace sbits;

// workspace: AllocState | keyU [N] | keyD [N] | trace [TRACE_CAP]
size_t sbits_alloc_ws_bytes(int64_t N)
{
    size_t b = sbits_align_up(sizeof(AllocState), 256);
    b += 2 * sbits_align_up((size_t)N * 8, 256);
    b += sbits_align_up((size_t)TRACE_CAP * sizeof(sbits_trace), 256);
    return b;
}

struct AllocWs { AllocState *st; u64 *keyU, *keyD; sbits_trace *tr; };
static AllocWs alloc_ws(void *ws, int64_t N)
{
    AllocWs w;
    char *p = static_cast<char *>(ws);
    w.st = reinterpret_cast<AllocState *>(p);
    p += sbits_align_up(sizeof(AllocState), 256);
    w.keyU = reinterpret_cast<u64 *>(p);
    p += sbits_align_up((size_t)N * 8, 256);
    w.keyD = reinterpret_cast<u64 *>(p);
    p += sbits_align_up((size_t)N * 8, 256);
    w.tr = reinterpret_cast<sbits_trace *>(p);
    return w;
}

template <bool STEP>
static void launch_search(hipStream_t sm, unsigned G, const AllocWs &w, int64_t N, const float *cost, const float *s_up,
                          const float *s_down, uint8_t *level, AllocResult *result, int only_if_aborted)
{
    auto *fn = (N + G - 1) / G <= (int64_t)AL_KPT * AL_THREADS ? &search_kernel<STEP, true> : &search_kernel<STEP, false>;
    hipLaunchKernelGGL(fn, dim3(G), dim3(AL_THREADS), 0, sm, w.st, cost, s_up, s_down, level, w.keyU, w.keyD, w.tr, result, SBITS_SPIN_LIMIT,
                       only_if_aborted);
}

static AllocHead start_head(const sbits_plan *plan, double avg_bits)
{
    AllocHead h;
    memset(&h, 0, sizeof h);
    h.N = plan->N;
    h.T = (long long)floor(avg_bits * (double)plan->N);
    h.K = plan->K;
    h.ceil_log2_n = ceil_log2_ll(plan->N);
    h.IB = h.ceil_log2_n > 0 ? h.ceil_log2_n : 1;
    for (int c = 0; c < MAX_CAND; ++c) h.bits[c] = c < plan->K ? plan->bits[c] : plan->bits[plan->K - 1];
    return h;
}

// The context's page-locked buffer, ready for the next result.
static int result_buffer(sbits_ctx *ctx, AllocResult **out)
{
    static_assert(sizeof(AllocResult) <= SBITS_PINNED_BYTES, "a result must fit the pinned buffer");
    if (!ctx->pinned) SBITS_HIP(ctx, hipHostMalloc(&ctx->pinned, SBITS_PINNED_BYTES, hipHostMallocDefault));
    *out = static_cast<AllocResult *>(ctx->pinned);
    (*out)->valid = 0;
    return SBITS_OK;
}

// A search that gave up and is not repeated (for tests) left nothing that may be used.
static int stop_if_aborted(sbits_ctx *ctx, const AllocState *st)
{
    AllocHead h;
    SBITS_HIP(ctx, hipMemcpyAsync(&h, &st->head, sizeof h, hipMemcpyDeviceToHost, ctx->stream));
    SBITS_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return h.aborted ? SBITS_ERR_INTERNAL : SBITS_OK;
}

int sbits_enqueue_allocate(sbits_plan *plan, const float *cost, double avg_bits, const sbits_params *prm, uint8_t *level, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    hipStream_t sm = ctx->stream;
    const int64_t N = plan->N;
    const int K = plan->K;
    if (avg_bits < (double)plan->bits[0]) return SBITS_ERR_INFEASIBLE_BUDGET;
    const AllocWs w = alloc_ws(ws, N);
    AllocResult *result;
    const int rc = result_buffer(ctx, &result);
    if (rc) return rc;

    AllocHead h0 = start_head(plan, avg_bits);
    h0.k = (long long)floor(prm->gamma0 * (double)N);
    h0.kmin = (long long)floor(prm->gammaT * (double)N);
    if (h0.k < 1) h0.k = 1;
    if (h0.kmin < 1) h0.kmin = 1;
    h0.max_iters = prm->max_iters;

    const bool all_max = avg_bits >= (double)plan->bits[K - 1];
    if (all_max) h0.l0 = K - 1;
    else if (prm->init_mode == 0) {
        const double fb = floor(avg_bits);
        for (int l = 0; l < K; ++l) if ((double)plan->bits[l] <= fb) h0.l0 = l;
    }
    h0.used = N * (long long)plan->bits[h0.l0];
    if (all_max) h0.done = 1;

    // The workgroups wait for each other.  Should the device be so full that they never run together, they
    // give up (see grid_sync) and one workgroup, which waits for nobody, does the search.
    const unsigned G = search_wgs(N, false, ctx->cus);
    hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(AL_THREADS), 0, sm, w.st, h0);
    launch_search<false>(sm, G, w, N, cost, nullptr, nullptr, level, result, 0);
    if (G > 1 && SBITS_SECOND_TRY) launch_search<false>(sm, 1, w, N, cost, nullptr, nullptr, level, result, 1);   // returns at once unless the first gave up
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_SECOND_TRY ? SBITS_OK : stop_if_aborted(ctx, w.st);
}

int sbits_finish_allocate(sbits_plan *plan, sbits_stats *host_stats, sbits_trace *host_trace, int64_t trace_cap, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    const AllocResult h = *static_cast<const AllocResult *>(ctx->pinned);
    if (!h.valid) return SBITS_ERR_INTERNAL;
    if (host_stats) {
        host_stats->iters = h.iters; host_stats->expansions = h.expansions;
        host_stats->swaps_ok = h.swaps_ok; host_stats->swaps_rej = h.swaps_rej;
        host_stats->k_final = h.k; host_stats->bits_used = h.bits_check; host_stats->bits_budget = h.budget;
        host_stats->cost_fixed = h.cost_fixed; host_stats->cost_shift = h.shift; host_stats->pad_ = 0;
    }
    if (host_trace && trace_cap > 0 && h.iters > 0) {
        int64_t nrec = h.iters < trace_cap ? h.iters : trace_cap;
        if (nrec > TRACE_CAP) nrec = TRACE_CAP;
        SBITS_HIP(ctx, hipMemcpyAsync(host_trace, alloc_ws(ws, plan->N).tr, (size_t)nrec * sizeof(sbits_trace), hipMemcpyDeviceToHost, ctx->stream));
        SBITS_HIP(ctx, hipStreamSynchronize(ctx->stream));
    }
    if (h.bits_check != h.used) return SBITS_ERR_INTERNAL;      // the loop's running total and a recount must agree
    return h.status;
}

// One step of Algorithm 2 on caller-supplied estimates.  Workspace as sbits_run_allocate.
int sbits_run_propose(sbits_plan *plan, const float *s_up, const float *s_down, const uint8_t *level_in,
                      double avg_bits, int64_t k, uint8_t *level_out, sbits_proposal *host_out, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    hipStream_t sm = ctx->stream;
    const int64_t N = plan->N;
    const AllocWs w = alloc_ws(ws, N);
    AllocResult *result = nullptr;                                   // (without a host output nothing is waited for)
    const int rc = host_out ? result_buffer(ctx, &result) : SBITS_OK;
    if (rc) return rc;
    AllocHead h = start_head(plan, avg_bits);
    h.k = k;
    // the start state travels as a kernel argument: nothing to keep alive, nothing to wait for
    hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(AL_THREADS), 0, sm, w.st, h);
    const unsigned G = search_wgs(N, true, ctx->cus);
    uint8_t *const lv = const_cast<uint8_t *>(level_in);             // (only read by the step)
    launch_search<true>(sm, G, w, N, nullptr, s_up, s_down, lv, result, 0);
    if (G > 1 && SBITS_SECOND_TRY) launch_search<true>(sm, 1, w, N, nullptr, s_up, s_down, lv, result, 1);   // returns at once unless the first gave up
    const unsigned grid = (unsigned)((N + 255) / 256 < 1024 ? (N + 255) / 256 : 1024);
    hipLaunchKernelGGL(step_apply_kernel, dim3(grid), dim3(256), 0, sm, (const AllocState *)w.st,
                       (const u64 *)w.keyU, (const u64 *)w.keyD, level_in, level_out);
    SBITS_HIP(ctx, hipGetLastError());
    if (host_out) {
        SBITS_HIP(ctx, hipStreamSynchronize(sm));
        const AllocResult r = *result;
        if (!r.valid) return SBITS_ERR_INTERNAL;
        host_out->kind = r.mode == MODE_EXPAND ? 1 : r.mode == MODE_ACCEPT ? 2 : 0;
        host_out->pad_ = 0;
        host_out->n_up = r.prop_up;
        host_out->n_dn = r.prop_dn;
        host_out->bits_before = r.used;
        host_out->bits_after = r.prop_after;
        host_out->bits_budget = r.budget;
    }
    return SBITS_OK;
}
