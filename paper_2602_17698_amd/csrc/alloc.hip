// Scalable greedy bitwidth search (paper Algorithm 2, relaxed step Eq. 5) on the
// block x bitwidth cost table, run on the device by ONE launch.
//
// Per iteration:
//   keys    : marginal cost change per bit of raising / lowering every block,
//             read off the table at the current levels (Alg. 2 line 5), encoded
//             as an ordered 32-bit word with the place of the block, [word : 32][N-1-index : 32],
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
// iteration), not bytes: the latency of barriers, LDS and exchanges, of scalar state in between, and the vector instructions on the
// keys.  G workgroups own a slice of the blocks each, in registers where it
// fits, and stay for the whole search; what they exchange (histograms, sums) goes through device-scope atomics
// into one of three rotating buffers, and every workgroup draws the same conclusions from the same sums.  An exchange shows by
// its values that it is complete, so nothing waits for the acknowledgement of what it added (see sel_rounds, team_sum).
// No fence: nothing else is shared, so no cache has to be written back or invalidated.  A round takes 1.7 us within
// one workgroup, 3 to 4 us with 7 to 26, 5 with 104, whose additions to the same bins take longer than the rest (512
// threads: 1024 spill and 256 leave the LDS atomics too few waves).
// Measured, whole searches (with a count of arrivals, 64-bit keys, one selection after the other, keys computed by the search's own
// workgroups -> now): 13 k blocks, 15 iterations 207 -> 183 us; 27 k, 15 iterations 346 -> 266; 107 k, 15 iterations 465 -> 355;
// 426 k, 15 iterations 428 -> 396; 336 blocks 87 -> 85; one proposal on 426 k blocks 67 -> 57, on 13 k 45 -> 37.
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
constexpr int AL_SUMS = 5;                    // values of one reduction, at most
constexpr int PREP_THREADS = 256, PREP_WGS = 512;
static_assert(PREP_WGS <= AL_THREADS, "a thread of the search reads what one workgroup of the preparation found");
constexpr int SEL_SETS = 2;                   // selections that go side by side
enum { UP, DOWN };                            // among the blocks that can be raised, among those that can be lowered

enum { MODE_NONE = 0, MODE_EXPAND = 1, MODE_ACCEPT = 2 };

struct AllocHead {
    long long N, T, k, kmin, used;
    int K, l0, max_iters, done, mode, min_step;
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
// gave_up: a word of its own, which the leader does not write: a workgroup may give up at the very last exchange.
struct AllocReport { AllocResult result; int pad_[16]; unsigned int gave_up; };
// One exchange between the workgroups; three of them take turns (see end_turn).
struct AllocXchg {
    unsigned long long hist[SEL_SETS][SEL_BINS];   // per bin: (sum of step widths << 32) | number of keys
    unsigned long long mark;                  // (workgroups that took part << 32) + the keys that they put into bins (see sel_rounds)
    unsigned long long part[2 * AL_SUMS];     // halves of sums, each with the number of workgroups that added theirs (see team_sum)
};
struct AllocState {
    AllocHead head;
    AllocXchg x[3];
    unsigned long long range[PREP_WGS][AL_SUMS];   // what each workgroup of the preparation found among its blocks
};

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
    int turn;                     // the exchange buffer in use
    int spin_limit;
    AllocReport *report;          // page-locked host memory, or null
    bool ok;                      // false: a wait was given up, leave
};

struct Sel { u64 tau; int n_sel, w_sel; };           // selected <=> key >= tau

// One selection: the longest prefix of the descending order of its keys with at most cnt_max keys and at most w_max step
// bits (neither negative).  The interval that the prefix ends in is one of words; when it has come down to a single word
// that several keys share, it is one of places among those (tie).  The same in every thread, in scalar registers: read from LDS
// it costs a round several hundred clocks.
struct Pick {
    unsigned from, last;                             // the interval, both ends in it
    unsigned base;                                   // bin of x: (x - base) >> shift; what is outside of the bins: the next one
    int shift;
    unsigned tie;                                    // the shared word, or 0
    int cnt_max, w_max;
    Sel r;                                           // keys and step bits above the interval; the threshold, once it has ended
};

constexpr int WS_SET = 16;                           // a wave's sums of set s: entry WS_SET * s + wave
struct AllocShared {
    alignas(16) u64 hist[SEL_SETS][SEL_BINS];
    u64 wave[2][64];                                 // sums of the waves (see sel_rounds)
    u64 mark;
    int live;
    int4 found[SEL_SETS];
    u64 sum[AL_SUMS], part[2][2 * AL_SUMS];
    int bits[MAX_CAND];
};

__device__ __forceinline__ AllocXchg *xchg(const Team &t) { return &t.st->x[t.turn]; }

// A wait between workgroups: how long one goes on polling.  Every wait is bounded: if a workgroup gets no place on the
// device, the others leave, each after its own wait, at this exchange or the next one; so do those that start later, at their
// first exchange that somebody is missing from.
__device__ __forceinline__ void give_up(Team &t)
{
    if (threadIdx.x == 0) {
        (void)__hip_atomic_fetch_add(&t.st->head.aborted, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t.report) t.report->gave_up = 1u;
    }
    t.ok = false;
}

// The end of a turn, after its values were read complete.  Whoever took part in it had read the buffer of the turn before: that one
// is cleared, and is in use again two turns later.  (Before a workgroup takes part in the next turn it waits for its clearing
// stores, so whoever finds the next turn complete finds that buffer clear.)
__device__ __forceinline__ void end_turn(Team &t)
{
    u64 *old = reinterpret_cast<u64 *>(&t.st->x[t.turn ? t.turn - 1 : 2]);
    constexpr int WORDS = (int)(sizeof(AllocXchg) / 8);
    const int per = (WORDS + t.G - 1) / t.G;
    for (int b = t.g * per + (int)threadIdx.x; b < min((t.g + 1) * per, WORDS); b += AL_THREADS) dev_store(&old[b], 0ull);
    t.turn = t.turn < 2 ? t.turn + 1 : 0;
}

// maximum or sum over the lanes of a wave, in lane 63 (the others hold parts of it)
template <bool MAX>
__device__ __forceinline__ u64 wave_reduce(u64 v)
{
    auto step = [&](auto ctrl, auto rows) {
        const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        const u64 o = (u64)hi << 32 | lo;            // (0 where there is no lane to take it from)
        v = MAX ? (o > v ? o : v) : v + o;
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1, 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2, 3
    return v;
}

// v[] of the whole workgroup to sum[] (LDS): maxima of the first NMAX, sums of the others
template <int NMAX, int NV>
__device__ __forceinline__ void block_reduce(u64 *sum, u64 (&v)[NV])
{
    static_assert(NV <= AL_SUMS, "slots");
    if (threadIdx.x < NV) sum[threadIdx.x] = 0ull;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const u64 o = q < NMAX ? wave_reduce<true>(v[q]) : wave_reduce<false>(v[q]);
        if ((threadIdx.x & 63) == 63 && o) {
            if (q < NMAX) atomicMax(&sum[q], o);
            else atomicAdd(&sum[q], o);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // (the clearing stores of the turn before, see end_turn)
    __syncthreads();
}

// Sums over all threads of all workgroups (mod 2^64); the same in every thread.  A sum travels in two halves of 32 bits, each
// in 48 bits below the number of workgroups (at most 256) that have added theirs: complete when that is all of them.
template <int NV>
__device__ __forceinline__ void team_sum(Team &t, AllocShared &sh, u64 (&v)[NV])
{
    __syncthreads();                                          // (the sums of the last time were read)
    block_reduce<0>(sh.sum, v);
    const int q = (int)threadIdx.x;
    if (t.G == 1) {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = uni(sh.sum[i]);
        return;
    }
    AllocXchg *x = xchg(t);
    if (q < 2 * NV) (void)__hip_atomic_fetch_add(&x->part[q], 1ull << 48 | (sh.sum[q >> 1] >> (q & 1 ? 32 : 0) & 0xffffffffull),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int left = t.spin_limit;
    for (int turn = 0;; turn ^= 1) {                          // (the buffers take turns: one barrier a poll)
        if (q < 2 * NV) sh.part[turn][q] = dev_load(&x->part[q]);
        __syncthreads();
        bool all = true;
        u64 h[2 * NV];
#pragma unroll
        for (int i = 0; i < 2 * NV; ++i) {
            h[i] = uni(sh.part[turn][i]);
            all = all && (int)(h[i] >> 48) == t.G;
        }
        if (all) {
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = (h[2 * i] & 0xffffffffffffull) + (h[2 * i + 1] << 32);
            break;
        }
        if (left-- <= 0) { give_up(t); return; }
    }
    end_turn(t);
}

// the smallest s with span >> s < SEL_BINS
__device__ __forceinline__ int bin_shift(unsigned span)
{
    const int len = 32 - __clz((int)(span | 1u));
    return len > SEL_DB ? len - SEL_DB : 0;
}

// Where a first round's bins are: they cover the words of the values above zero, where nearly all keys lie; the outermost bins
// hold what is below and above.  none: no value is above zero.
struct Bins { unsigned lo, hi, base; int shift; };
__device__ __forceinline__ Bins bins_over(unsigned lo, unsigned hi)
{
    const unsigned span = hi > lo ? hi - lo : 0u, wide = span + 2 * (span >> (SEL_DB - 1)) + 2u;    // (two bins are the outermost)
    Bins b;
    b.lo = lo; b.hi = hi;
    b.shift = bin_shift(wide < span ? ~0u : wide);
    b.base = lo > 1u << b.shift ? lo - (1u << b.shift) : 0u;
    return b;
}
struct Ranges { Bins up, down; };                     // of keyU, of keyD

// A workgroup's blocks: the words of their two keys (0: cannot be raised / lowered; in 32 bits, because a round is bound by
// the vector instructions on them: with 64-bit keys a round of one workgroup took 3 us, 2 of them here), the widths of the two steps, four bits each, and
// their levels.  A thread owns blocks n0 + tid,
// n0 + tid + AL_THREADS, ... and nobody else touches what belongs to them.  RES: it holds all of them (at most
// AL_KPT) in registers; otherwise they live in memory and come in AL_KPT at a time.
struct Batch { unsigned ku[AL_KPT], kd[AL_KPT], su, sd; int lv[AL_KPT]; };
__device__ __forceinline__ unsigned width_of(unsigned packed, int q) { return packed >> (4 * q) & 15u; }
__device__ __forceinline__ void set_width(unsigned &packed, int q, unsigned w) { packed = (packed & ~(15u << (4 * q))) | w << (4 * q); }
template <bool RES>
struct Slice {
    Batch reg;                    // RES
    u64 *mu, *md;                 // [N] in the workspace: word << 32 | width
    uint8_t *level;
    int n0, n1;
    int used;                     // RES: slots of a thread that hold blocks

    // f(first block of the batch, batch, slots): block u of it is first + u * AL_THREADS, there if < n1 (else its keys are 0).
    // What f changes is kept (WR) in all arrays.  need_kd: f looks at keyD (from memory it is half of the bytes).
    template <bool LV, bool WR, class F>
    __device__ __forceinline__ void visit(F &&f, bool need_kd = true)
    {
        if constexpr (RES) {
            f(n0 + (int)threadIdx.x, reg, used);
        } else {
            for (int i0 = n0 + (int)threadIdx.x; i0 < n1; i0 += AL_KPT * AL_THREADS) {
                Batch b;
                b.su = b.sd = 0u;
                u64 w[AL_KPT];
#pragma unroll
                for (int u = 0; u < AL_KPT; ++u) {
                    const int i = i0 + u * AL_THREADS;
                    w[u] = i < n1 ? mu[i] : 0ull;
                    b.lv[u] = LV && i < n1 ? (int)level[i] : 0;
                }
#pragma unroll
                for (int u = 0; u < AL_KPT; ++u) { b.ku[u] = (unsigned)(w[u] >> 32); set_width(b.su, u, (unsigned)w[u]); b.kd[u] = 0u; }
                if (need_kd) {
#pragma unroll
                    for (int u = 0; u < AL_KPT; ++u) {
                        const int i = i0 + u * AL_THREADS;
                        w[u] = i < n1 ? md[i] : 0ull;
                    }
#pragma unroll
                    for (int u = 0; u < AL_KPT; ++u) { b.kd[u] = (unsigned)(w[u] >> 32); set_width(b.sd, u, (unsigned)w[u]); }
                }
                f(i0, b, AL_KPT);
                if constexpr (WR) store(i0, b);
            }
        }
    }
    __device__ __forceinline__ void store(int i0, const Batch &b)
    {
#pragma unroll
        for (int u = 0; u < AL_KPT; ++u) {
            const int i = i0 + u * AL_THREADS;
            if (i < n1) {
                mu[i] = (u64)b.ku[u] << 32 | width_of(b.su, u);
                md[i] = (u64)b.kd[u] << 32 | width_of(b.sd, u);
                level[i] = (uint8_t)b.lv[u];
            }
        }
    }
    // the blocks for the first time, from memory
    __device__ __forceinline__ void load(int lv)
    {
        u64 a[AL_KPT], b[AL_KPT];
#pragma unroll
        for (int u = 0; u < AL_KPT; ++u) {
            const int i = n0 + (int)threadIdx.x + u * AL_THREADS;
            a[u] = i < n1 ? mu[i] : 0ull;
            b[u] = i < n1 ? md[i] : 0ull;
        }
        reg.su = reg.sd = 0u;
#pragma unroll
        for (int u = 0; u < AL_KPT; ++u) {
            reg.ku[u] = (unsigned)(a[u] >> 32); reg.kd[u] = (unsigned)(b[u] >> 32); reg.lv[u] = lv;
            set_width(reg.su, u, (unsigned)a[u]);
            set_width(reg.sd, u, (unsigned)b[u]);
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

// A selection at its start: among the keys of words from and above (from >= 1: no key that says that there is no step).
__device__ __forceinline__ Pick pick(unsigned from, const Bins &b, int cnt_max, int w_max)
{
    return Pick{from, ~0u, b.base, b.shift, 0u, cnt_max, w_max, {~0ull, 0, 0}};
}

// The selection after the round in which its prefix ended in bin b (-1: every key fitted), with ac keys of aw step bits above
// and n keys in it.  Returns whether it has ended.
__device__ __forceinline__ bool narrow(Pick &p, int b, int n, int ac, int aw, int N)
{
    p.r.n_sel = ac;
    p.r.w_sel = aw;
    if (b < 0) {
        p.r.tau = p.tie ? (u64)p.tie << 32 | p.from : (u64)p.from << 32;
        return true;
    }
    const unsigned begin = p.base + ((unsigned)b << p.shift), end = begin + ((1u << p.shift) - 1u);    // (it holds a key: only its end may be past 32 bits)
    if (b < SEL_BINS - 1 && end >= begin && end < p.last) p.last = end;
    if (b > 0 && begin > p.from) p.from = begin;
    if (n == 1 || (p.tie && p.from == p.last)) {     // one key that does not fit: the prefix ends above it
        p.r.tau = p.tie ? (u64)p.tie << 32 | (p.last + 1u) : p.last == ~0u ? ~0ull : (u64)(p.last + 1u) << 32;
        return true;
    }
    if (p.from == p.last) {                          // several keys of one word: their places decide
        p.tie = p.from;
        p.from = 0u;
        p.last = (unsigned)(N - 1);
    }
    p.base = p.from;
    p.shift = bin_shift(p.last - p.from);
    return false;
}

__device__ __forceinline__ u64 key_at(unsigned word, int place) { return (u64)word << 32 | (unsigned)place; }

// The selections p of `open` (a bit each), side by side: UP among the keyU, DOWN among the keyD of the blocks outside the set
// keyU >= excl.  Each round splits a selection's interval into bins and goes on with the bin in which the prefix ends,
// until that bin holds one key.  sh.hist is all zero before and after.
//
// The exchange.  Every workgroup adds its bins and, without waiting for that, to `mark` how many keys they hold.  One thread polls `mark`
// until all workgroups have said so; then the bins are read until they hold as many as it says.  (All threads polling the bins, or
// a mark from every wave, are in the way of the additions: 104 workgroups 775 us against 425.)
template <bool RES>
__device__ __forceinline__ void sel_rounds(Team &t, AllocShared &sh, Slice<RES> &own, Pick (&p)[SEL_SETS], unsigned open, u64 excl, int N)
{
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
#pragma unroll 1
    while (open) {
        int live = 0;                                // keys put into bins (of this wave: the first lane's)
        own.template visit<false, false>([&](int i0, const Batch &bt, int slots) {
            static_for<0, SEL_SETS>([&](auto is) {
                constexpr int s = decltype(is)::value;
                if (!(open & 1u << s)) return;
                const unsigned span = p[s].last - p[s].from;
#pragma unroll
                for (int q = 0; q < AL_KPT; ++q) {
                    if (q >= slots) break;
                    const int place = N - 1 - (i0 + q * AL_THREADS);
                    unsigned x = s == DOWN ? bt.kd[q] : bt.ku[q];
                    if (s == DOWN && excl != ~0ull && key_at(bt.ku[q], place) >= excl) x = 0u;
                    bool in = x - p[s].from <= span;
                    if (p[s].tie) {
                        in = x == p[s].tie && (unsigned)place - p[s].from <= span;
                        x = (unsigned)place;
                    }
                    live += __popcll(__ballot(in));
                    if (in) {
                        const unsigned n = __builtin_elementwise_sub_sat(x, p[s].base) >> p[s].shift;
                        const int b = (int)(n < SEL_BINS ? n : SEL_BINS - 1);
                        atomicAdd(&sh.hist[s][SEL_BINS - 1 - b], (u64)width_of(s == DOWN ? bt.sd : bt.su, q) << 32 | 1ull);   // descending: the top bin first
                    }
                }
            });
        }, open & 1u << DOWN);
        AllocXchg *const x = xchg(t);
        if (t.G > 1) {
            if (lane == 0 && live) atomicAdd(&sh.live, live);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // (the clearing stores of the turn before)
        }
        __syncthreads();
        u64 v[SEL_SETS][AL_BPT];                     // a thread has AL_BPT consecutive bins
        static_for<0, SEL_SETS>([&](auto is) {
            constexpr int s = decltype(is)::value;
            if (!(open & 1u << s)) return;
#pragma unroll
            for (int q = 0; q < AL_BPT; ++q) {
                u64 &b = sh.hist[s][tid * AL_BPT + q];
                v[s][q] = b;
                b = 0ull;
                if (t.G > 1 && v[s][q])
                    (void)__hip_atomic_fetch_add(&x->hist[s][tid * AL_BPT + q], v[s][q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        });
        int pc[SEL_SETS], pw[SEL_SETS];              // sums over the bins above (at most 2^24 keys of width <= 8: below 2^31)
        int left = t.spin_limit, all = 0;
        if (t.G > 1) {
            if (tid == 0) {
                (void)__hip_atomic_fetch_add(&x->mark, 1ull << 32 | (u64)(unsigned)sh.live, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh.live = 0;
                u64 m;
                while ((int)((m = dev_load(&x->mark)) >> 32) != t.G && left-- > 0) __builtin_amdgcn_s_sleep(1);
                sh.mark = m;
            }
            __syncthreads();
            const u64 m = uni(sh.mark);
            if ((int)(m >> 32) != t.G) { give_up(t); return; }
            all = (int)(unsigned)m;
            left = t.spin_limit;
        }
#pragma unroll 1
        for (int turn = 0;; turn ^= 1) {             // (the waves' sums take turns in two buffers: one barrier a read)
            if (t.G > 1) {
                static_for<0, SEL_SETS>([&](auto is) {
                    constexpr int s = decltype(is)::value;
                    if (!(open & 1u << s)) return;
#pragma unroll
                    for (int q = 0; q < AL_BPT; ++q) v[s][q] = dev_load(&x->hist[s][tid * AL_BPT + q]);
                });
            }
            static_for<0, SEL_SETS>([&](auto is) {
                constexpr int s = decltype(is)::value;
                if (!(open & 1u << s)) return;
                int c = 0, w = 0;
#pragma unroll
                for (int q = 0; q < AL_BPT; ++q) { c += (int)v[s][q]; w += (int)(v[s][q] >> 32); }
                const int ic = (int)wave_prefix((unsigned)c), iw = (int)wave_prefix((unsigned)w);
                pc[s] = ic - c;
                pw[s] = iw - w;
                if (lane == 63) sh.wave[turn][WS_SET * s + wave] = (u64)(unsigned)iw << 32 | (unsigned)ic;
            });
            __syncthreads();
            // lanes 0 .. 7 of a row of 16 have the sums of set (row); a prefix over them
            const u64 e = sh.wave[turn][lane];
            const int ec = (int)e, ew = (int)(e >> 32);
            int sc = ec, sw = ew;
            auto step = [&](auto ctrl) {
                sc += __builtin_amdgcn_update_dpp(0, sc, decltype(ctrl)::value, 0xf, 0xf, true);
                sw += __builtin_amdgcn_update_dpp(0, sw, decltype(ctrl)::value, 0xf, 0xf, true);
            };
            step(std::integral_constant<int, 0x111>{});               // row_shr:1, 2, 4
            step(std::integral_constant<int, 0x112>{});
            step(std::integral_constant<int, 0x114>{});
            int sum = 0;
            static_for<0, SEL_SETS>([&](auto is) {
                constexpr int s = decltype(is)::value;
                if (!(open & 1u << s)) return;
                pc[s] += __builtin_amdgcn_readlane(sc - ec, WS_SET * s + wave);
                pw[s] += __builtin_amdgcn_readlane(sw - ew, WS_SET * s + wave);
                sum += __builtin_amdgcn_readlane(sc, WS_SET * s + AL_WAVES - 1);
            });
            if (t.G == 1 || sum == all) break;
            if (left-- <= 0) { give_up(t); return; }
        }
        // The sums only grow downwards, so the first bin that does not fit whole is the one that does not fit while
        // everything above it does; it ends the prefix.
        static_for<0, SEL_SETS>([&](auto is) {
            constexpr int s = decltype(is)::value;
            if (!(open & 1u << s)) return;
            int ac = p[s].r.n_sel + pc[s], aw = p[s].r.w_sel + pw[s];
#pragma unroll
            for (int q = 0; q < AL_BPT; ++q) {
                const int n = (int)v[s][q], ic = ac + n, iw = aw + (int)(v[s][q] >> 32);
                const bool fits = ic <= p[s].cnt_max && iw <= p[s].w_max;
                if (n && !fits && ac <= p[s].cnt_max && aw <= p[s].w_max) sh.found[s] = make_int4(SEL_BINS - 1 - (tid * AL_BPT + q), n, ac, aw);
                else if (q == AL_BPT - 1 && tid == AL_THREADS - 1 && fits) sh.found[s] = make_int4(-1, 0, ic, iw);
                ac = ic; aw = iw;
            }
        });
        __syncthreads();
        int4 f[SEL_SETS];
        static_for<0, SEL_SETS>([&](auto is) {
            constexpr int s = decltype(is)::value;
            if (open & 1u << s) f[s] = sh.found[s];
        });
        if (t.G > 1) end_turn(t);
        static_for<0, SEL_SETS>([&](auto is) {
            constexpr int s = decltype(is)::value;
            if (open & 1u << s && narrow(p[s], uni(f[s].x), uni(f[s].y), uni(f[s].z), uni(f[s].w), N)) open &= ~(1u << s);
        });
    }
}

__device__ __forceinline__ void trace_write(sbits_trace *tr, int it, int kind, long long k, long long n_up, long long n_dn,
                                            long long p_up, long long p_dn, long long before, long long after, long long delta)
{
    if (it >= TRACE_CAP) return;
    sbits_trace &t = tr[it];
    t.kind = kind; t.pad_ = 0; t.k = k; t.n_up = n_up; t.n_dn = n_dn; t.p_up = p_up; t.p_dn = p_dn;
    t.bits_before = before; t.bits_after = after; t.delta_fixed = delta;
}

// 0 is no word of a key: it says that there is no step
__device__ __forceinline__ unsigned some(unsigned word) { return word ? word : 1u; }

// The sets of one iteration of Algorithm 2.  e: the expansion (not tried without slack): the first k blocks by
// keyU with a value above zero that fit the slack.  If it is empty, the balanced swap: u = the first h by keyU,
// d = the first h by keyD outside u, u2 = the longest prefix of u whose step bits fit the slack plus the bits d
// frees.
// u and d go side by side, d as if u took none of its blocks: what a raise gains the least is what a lowering costs the
// least, so the two hardly ever meet.  The caller counts the blocks that are in both and, if there are any, asks again with
// apart = u's threshold.
// STEP: the levels are the caller's and may be over budget; the search's own never are.
struct Sets { Sel e, u, d, u2; };
template <bool STEP, bool RES>
__device__ __forceinline__ void choose_sets(Team &t, AllocShared &sh, Slice<RES> &own, long long k, long long slack, int min_step,
                                            const Ranges &rg, int N, u64 apart, Sets &o)
{
    const int INF = 0x7fffffff;
    auto clip = [](long long v) { return (int)(v < -1 ? -1 : v > INF ? INF : v); };
    const int h = k / 2 < 1 ? 1 : clip(k / 2);
    Pick p[SEL_SETS];
    p[UP] = pick(1u, rg.up, h, INF);
    p[DOWN] = pick(1u, rg.down, h, INF);
    enum { EXPAND, BOTH, AGAIN, FIT };
    int phase = BOTH;
    unsigned open = 1u << UP | 1u << DOWN;
    if (apart != ~0ull) {
        phase = AGAIN;
        open = 1u << DOWN;
    } else {
        o.e = o.u = o.d = o.u2 = Sel{~0ull, 0, 0};
        if (slack >= min_step && rg.up.hi) {         // (else no step fits, or none is worth taking)
            phase = EXPAND;
            open = 1u << UP;
            p[UP] = pick(0x80000001u, rg.up, clip(k), clip(slack));  // (values above +0)
        }
    }
#pragma unroll 1
    for (;;) {                                       // (one copy of the rounds: inlined several times they spill)
        sel_rounds(t, sh, own, p, open, apart, N);
        if (!t.ok) return;
        if (phase == EXPAND) {
            o.e = p[UP].r;
            if (o.e.n_sel > 0) return;
            phase = BOTH;
            open = 1u << UP | 1u << DOWN;
            p[UP] = pick(1u, rg.up, h, INF);
            continue;
        }
        if (phase == FIT) { o.u2 = p[UP].r; return; }
        if (phase == BOTH) o.u = p[UP].r;
        o.d = p[DOWN].r;
        o.u2 = o.u;
        if (o.u.w_sel <= slack + o.d.w_sel) return;                  // all of u fits
        if constexpr (STEP)
            if (slack + o.d.w_sel < 0) { o.u2 = Sel{~0ull, 0, 0}; return; }   // over by more than d frees: nothing of u does
        phase = FIT;
        open = 1u << UP;
        const unsigned from = (unsigned)(o.u.tau >> 32);              // u has no keys below these words
        p[UP] = pick(from, bins_over(from > rg.up.lo ? from : rg.up.lo, rg.up.hi), h, clip(slack + o.d.w_sel));
    }
}

// The words of the values above zero, from the largest one and the complement of the smallest one: of keyU, and of keyD, which
// are complements.  0 to 0 if there is none.
__device__ __forceinline__ Ranges value_ranges(u64 omax, u64 omin_inv)
{
    return Ranges{bins_over(omax ? ~(unsigned)omin_inv : 0u, (unsigned)omax), bins_over(omax ? ~(unsigned)omax : 0u, (unsigned)omin_inv)};
}

// Where a search begins, with every CU at work (computed by the search's few workgroups themselves it took 20 us for 107 k blocks):
// keys of blocks first, first + stride, ... at level l0, and of all gains in their rows of the table the largest and the
// smallest inverted above zero, and the largest entry.
__device__ __forceinline__ void table_keys(const float *__restrict__ cost, int N, int K, const int *bits, int l0, int first, int stride,
                                           uint8_t *level, u64 *__restrict__ keyU, u64 *__restrict__ keyD, u64 (&red)[3])
{
    for (int i = first; i < N; i += stride) {
        float c[MAX_CAND];
#pragma unroll
        for (int l = 0; l < MAX_CAND; ++l) c[l] = l < K ? cost[(int64_t)i * K + l] : 0.0f;
        u64 ku = 0ull, kd = 0ull;
#pragma unroll
        for (int l = 0; l < MAX_CAND; ++l) {
            if (l >= K) continue;
            if (c[l] > 0.0f) red[2] = max(red[2], (u64)__float_as_uint(c[l]));
            if (l) {
                const unsigned step = (unsigned)(bits[l] - bits[l - 1]), o = ord_f32((c[l - 1] - c[l]) / (float)step);
                if (o > 0x80000000u) { red[0] = max(red[0], (u64)o); red[1] = max(red[1], (u64)~o); }
                if (l == l0 + 1) ku = (u64)some(o) << 32 | step;
                if (l == l0) kd = (u64)some(~o) << 32 | step;
            }
        }
        keyU[i] = ku;
        keyD[i] = kd;
        level[i] = (uint8_t)l0;
    }
}
// The same for a step on the caller's estimates at the caller's levels: largest and smallest inverted of s_up above zero, of
// s_down, and the bits in use.
__device__ __forceinline__ void step_keys(const float *__restrict__ s_up, const float *__restrict__ s_down, const uint8_t *level, int N, int K,
                                          const int *bits, int first, int stride, u64 *__restrict__ keyU, u64 *__restrict__ keyD, u64 (&red)[5])
{
#pragma unroll 4
    for (int i = first; i < N; i += stride) {
        const int l = min((int)level[i], K - 1);
        const float up = s_up[i], dn = s_down[i];
        red[4] += (u64)bits[l];
        u64 ku = 0, kd = 0;
        if (l < K - 1) {
            const unsigned int o = ord_f32(up);
            ku = (u64)some(o) << 32 | (unsigned)(bits[l + 1] - bits[l]);
            if (o > 0x80000000u) { red[0] = max(red[0], (u64)o); red[1] = max(red[1], (u64)~o); }
        }
        if (l > 0) {
            const unsigned int o = ord_f32(dn);
            kd = (u64)some(~o) << 32 | (unsigned)(bits[l] - bits[l - 1]);
            if (o > 0x80000000u) { red[2] = max(red[2], (u64)o); red[3] = max(red[3], (u64)~o); }
        }
        keyU[i] = ku;
        keyD[i] = kd;
    }
}

// Ahead of the search: its start state (from a kernel argument: no host buffer has to outlive the call), clear exchange
// buffers, keys and their ranges.
template <bool STEP>
__global__ __launch_bounds__(PREP_THREADS)
void prepare_kernel(AllocState *st, AllocHead head, const float *__restrict__ cost, const float *__restrict__ s_up,
                    const float *__restrict__ s_down, uint8_t *level, u64 *__restrict__ keyU, u64 *__restrict__ keyD)
{
    __shared__ u64 sum[AL_SUMS];
    __shared__ int bits[MAX_CAND];
    const int tid = (int)threadIdx.x, at = (int)blockIdx.x * PREP_THREADS + tid, all = (int)gridDim.x * PREP_THREADS;
    if (at == 0) st->head = head;
    u64 *j = reinterpret_cast<u64 *>(st->x);
    for (int i = at; i < (int)(sizeof(st->x) / 8); i += all) j[i] = 0ull;
    if (tid < MAX_CAND) bits[tid] = head.bits[tid];
    __syncthreads();
    if constexpr (STEP) {
        u64 red[5] = {0, 0, 0, 0, 0};
        step_keys(s_up, s_down, level, (int)head.N, head.K, bits, at, all, keyU, keyD, red);
        block_reduce<4>(sum, red);
    } else {
        u64 red[3] = {0, 0, 0};
        table_keys(cost, (int)head.N, head.K, bits, head.l0, at, all, level, keyU, keyD, red);
        block_reduce<3>(sum, red);
    }
    if (tid < (STEP ? 5 : 3)) st->range[blockIdx.x][tid] = sum[tid];
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
                   sbits_trace *tr, AllocReport *report, int n_ranges, int spin_limit, int only_if_aborted)
{
    __shared__ AllocShared sh;
    const int tid = (int)threadIdx.x;
    if (only_if_aborted && !st->head.aborted) return;
    Team t;
    t.st = st; t.G = (int)gridDim.x; t.g = (int)blockIdx.x; t.turn = 0; t.spin_limit = spin_limit; t.report = report; t.ok = true;
    const int N = uni((int)st->head.N), K = uni(st->head.K), per = (N + t.G - 1) / t.G;      // (N <= 2^24)
    const long long T = st->head.T;
    for (int b = tid; b < SEL_SETS * SEL_BINS; b += AL_THREADS) sh.hist[0][b] = 0ull;
    if (tid == 0) sh.live = 0;
    if (tid < MAX_CAND) sh.bits[tid] = st->head.bits[tid];
    constexpr int NRED = STEP ? 5 : 3, NMAX = STEP ? 4 : 3;
    u64 red[NRED] = {};
    if (tid < n_ranges) {
#pragma unroll
        for (int q = 0; q < NRED; ++q) red[q] = st->range[tid][q];
    }
    block_reduce<NMAX>(sh.sum, red);
#pragma unroll
    for (int q = 0; q < NRED; ++q) red[q] = uni(sh.sum[q]);
    const int *bits = sh.bits;
    const bool lead = blockIdx.x == 0 && tid == AL_THREADS - 64;     // (of the last wave: it is waited for the least)
    const int min_step = uni(st->head.min_step), l0 = uni(st->head.l0);
    long long used = st->head.used, k = st->head.k;
    if constexpr (!STEP) {
        if (only_if_aborted) {                       // keys and levels as they were before the first try
            u64 again[3] = {0, 0, 0};
            table_keys(cost, N, K, bits, l0, tid, AL_THREADS, level, keyU, keyD, again);
            __syncthreads();
        }
    }
    Slice<RES> own;
    own.mu = keyU; own.md = keyD; own.level = level;
    own.n0 = min(N, per * t.g);
    own.n1 = min(N, own.n0 + per);
    own.used = (own.n1 - own.n0 + AL_THREADS - 1) / AL_THREADS;
    if constexpr (RES) own.load(l0);
    Ranges rg;
    if constexpr (STEP) {
        rg.up = value_ranges(red[0], red[1]).up;
        rg.down = value_ranges(red[2], red[3]).down;
        used = (long long)red[4];
        Sets o;
        const Sel &e = o.e, &u = o.u, &d = o.d, &u2 = o.u2;
        for (u64 apart = ~0ull;;) {
            choose_sets<STEP>(t, sh, own, k, T - used, min_step, rg, N, apart, o);
            if (!t.ok) return;
            if (e.n_sel > 0 || apart != ~0ull) break;
            u64 both[1] = {0};
            own.template visit<false, false>([&](int i0, const Batch &bt, int) {
#pragma unroll
                for (int q = 0; q < AL_KPT; ++q) {
                    const int place = N - 1 - (i0 + q * AL_THREADS);
                    both[0] += key_at(bt.kd[q], place) >= d.tau && key_at(bt.ku[q], place) >= u.tau;
                }
            });
            team_sum(t, sh, both);
            if (!t.ok) return;
            if (!both[0]) break;
            apart = u.tau;
        }
        // (a swap is a proposal: the caller accepts or rejects it)
        const int mode = e.n_sel > 0 ? MODE_EXPAND : u2.n_sel > 0 && d.n_sel > 0 ? MODE_ACCEPT : MODE_NONE;
        if (lead) {
            AllocHead &hd = st->head;
            hd.mode = mode;
            hd.tauE = e.tau; hd.tauU = u.tau; hd.tauD = d.tau; hd.tauU2 = u2.tau;
            if (report) {
                AllocResult r = {};
                r.used = used; r.budget = T;
                r.mode = mode;
                r.prop_up = mode == MODE_EXPAND ? e.n_sel : mode == MODE_ACCEPT ? u2.n_sel : 0;
                r.prop_dn = mode == MODE_ACCEPT ? d.n_sel : 0;
                r.prop_after = used + (mode == MODE_EXPAND ? e.w_sel : mode == MODE_ACCEPT ? u2.w_sel - d.w_sel : 0);
                r.valid = 1;
                report->result = r;
            }
        }
    } else {
        int shift = 0;
        if (red[2]) {
            const unsigned int b = (unsigned int)red[2];
            const int e = (int)(b >> 23);
            const int ilog = e ? e - 127 : (31 - __clz((int)(b & 0x7fffffu))) - 149;
            shift = 61 - st->head.ceil_log2_n - (ilog + 1);
        }
        rg = value_ranges(red[0], red[1]);
        const long long kmin = st->head.kmin;
        const int max_iters = st->head.max_iters;
        int iters = 0, expansions = 0, swaps_ok = 0, swaps_rej = 0, status = SBITS_OK;
        bool done = st->head.done != 0;
        // The blocks that way(keyU, keyD) moves by +1 or -1 get their new level and keys.  What it cost to leave the old level
        // is, complemented, the key of the way back; the other key is read off the table.  (All loads of a batch are
        // requested before any is used.)
        struct Moves { int by[AL_KPT]; float a[AL_KPT], b[AL_KPT]; };
        auto ask = [&](int i0, const Batch &bt, Moves &m, auto way) {
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const int i = i0 + q * AL_THREADS;
                m.by[q] = i < own.n1 ? way(key_at(bt.ku[q], N - 1 - i), key_at(bt.kd[q], N - 1 - i)) : 0;
                m.a[q] = m.b[q] = 0.0f;
                if (m.by[q]) {
                    const int from = bt.lv[q] + (m.by[q] > 0 ? 1 : -2);              // the next step from there
                    if (from >= 0 && from < K - 1) {
                        const float *c = cost + (int64_t)i * K + from;
                        m.a[q] = c[0];
                        m.b[q] = c[1];
                    }
                }
            }
        };
        auto apply = [&](Batch &bt, const Moves &m) {
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q)
                if (m.by[q]) {
                    const bool up = m.by[q] > 0;
                    const int from = bt.lv[q] + (up ? 1 : -2);
                    unsigned word = 0u, step = 0u;
                    if (from >= 0 && from < K - 1) {
                        step = (unsigned)(bits[from + 1] - bits[from]);
                        const unsigned o = ord_f32((m.a[q] - m.b[q]) / (float)step);
                        word = some(up ? o : ~o);
                    }
                    const unsigned back = some(~(up ? bt.ku[q] : bt.kd[q])), wide = width_of(up ? bt.su : bt.sd, q);
                    bt.ku[q] = up ? word : back;
                    bt.kd[q] = up ? back : word;
                    set_width(bt.su, q, up ? step : wide);
                    set_width(bt.sd, q, up ? wide : step);
                    bt.lv[q] += m.by[q];
                }
        };
        auto move = [&](auto way) {
            own.template visit<true, true>([&](int i0, Batch &bt, int) {
                Moves m;
                ask(i0, bt, m, way);
                apply(bt, m);
            });
        };
        Sets o;
        const Sel &e = o.e, &u = o.u, &d = o.d, &u2 = o.u2;
        u64 apart = ~0ull;
        while (!done) {
            choose_sets<STEP>(t, sh, own, k, T - used, min_step, rg, N, apart, o);
            if (!t.ok) return;
            if (e.n_sel > 0) {
                move([&](u64 ku, u64) { return ku >= e.tau ? 1 : 0; });
                if (lead) trace_write(tr, iters, 0, k, e.n_sel, 0, e.n_sel, 0, used, used + e.w_sel, 0);
                used += e.w_sel;
                ++expansions;
            } else {
                u64 lg[3] = {0, 0, 0};               // the swap's loss and gain; blocks that both sets hold
                auto way = [&](u64 ku, u64 kd) { return ku >= u2.tau ? 1 : (kd >= d.tau && !(ku >= u.tau)) ? -1 : 0; };
                own.template visit<true, false>([&](int i0, const Batch &bt, int) {
                    int by[AL_KPT];
                    float hi[AL_KPT], lo[AL_KPT];    // the table entries below and above the step
#pragma unroll
                    for (int q = 0; q < AL_KPT; ++q) {
                        const int i = i0 + q * AL_THREADS;
                        const u64 ku = key_at(bt.ku[q], N - 1 - i), kd = key_at(bt.kd[q], N - 1 - i);
                        by[q] = i < own.n1 ? way(ku, kd) : 0;
                        lg[2] += i < own.n1 && kd >= d.tau && ku >= u.tau;
                        hi[q] = lo[q] = 0.0f;
                        if (by[q]) {
                            const float *c = cost + (int64_t)i * K + bt.lv[q] + (by[q] > 0 ? 0 : -1);
                            hi[q] = c[0];
                            lo[q] = c[1];
                        }
                    }
#pragma unroll
                    for (int q = 0; q < AL_KPT; ++q)
                        if (by[q]) lg[by[q] > 0] += (u64)fx(hi[q] - lo[q], shift);
                });
                Moves m;                             // (what the swap will need of the table if it is accepted, asked for in good time)
                if constexpr (RES) ask(own.n0 + tid, own.reg, m, way);
                team_sum(t, sh, lg);
                if (!t.ok) return;
                if (lg[2] && apart == ~0ull) {       // d has blocks of u: it is chosen again, outside u
                    apart = u.tau;
                    continue;
                }
                apart = ~0ull;
                const long long delta = (long long)(lg[0] - lg[1]);
                if (u2.n_sel > 0 && d.n_sel > 0 && delta < 0) {
                    if constexpr (RES) apply(own.reg, m);
                    else move(way);
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
        own.template visit<true, false>([&](int i0, const Batch &bt, int) {
            float c[AL_KPT];
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q) {
                const int i = i0 + q * AL_THREADS;
                c[q] = 0.0f;
                if (i < own.n1) {
                    c[q] = cost[(int64_t)i * K + bt.lv[q]];
                    if constexpr (RES) level[i] = (uint8_t)bt.lv[q];
                }
            }
#pragma unroll
            for (int q = 0; q < AL_KPT; ++q)
                if (i0 + q * AL_THREADS < own.n1) {
                    fin[0] += (u64)fx(c[q], shift);
                    fin[1] += (u64)bits[bt.lv[q]];
                }
        });
        team_sum(t, sh, fin);
        if (!t.ok) return;
        if (lead) {
            AllocResult r = {};
            r.used = used; r.k = k; r.budget = T; r.shift = shift; r.status = status;
            r.iters = iters; r.expansions = expansions; r.swaps_ok = swaps_ok; r.swaps_rej = swaps_rej;
            r.cost_fixed = (long long)fin[0]; r.bits_check = (long long)fin[1];
            r.valid = 1;
            report->result = r;
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
    const long long N = hd.N;          // (the widths that the keys end in in memory make way for the blocks' places)
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
        const u64 ku = key_at((unsigned)(keyU[i] >> 32), (int)(N - 1 - i)), kd = key_at((unsigned)(keyD[i] >> 32), (int)(N - 1 - i));
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

// ---- at most 64 blocks: one wave, a block a lane ------------------------------------------------
// The same search or step, by itself: no launch before it and none after it.  A round of the search above is the latency of barriers
// and LDS however few the keys are, and a selection is a round or more; here a lane counts the keys above its own and adds up their
// step bits, six instructions a key, and has every set that can be a prefix of that order.  What bounds it is the issue of one wave.
// Measured, calls on three candidates (two launches of a workgroup -> one of a wave): 16 blocks, 7 iterations 69.9 -> 24.4 us; 64 blocks,
// 26 iterations 188 -> 100; a step 26 -> 17; the kernels of a search of a 512 x 512 matrix 27 to 49 and 4 -> 7 to 12.  The line lies
// where a lane has one block: an iteration takes 1.5 us for 16 blocks and 3.3 for 64, 6.4 in the rounds, and with two blocks a lane
// it would be four times the work.
constexpr int WAVE_BLOCKS = 64;

struct Ranked { int rank, bits; };                   // keys above the lane's own; step bits of those and its own
// Keys of word 0 take no part (and their lanes' results say nothing).
__device__ __forceinline__ Ranked rank_keys(unsigned word, unsigned width, int N)
{
    const unsigned one = 1u << 16 | width;           // (64 widths of at most 8 stay below 2^16)
    const u64 key = key_at(word, WAVE_BLOCKS - 1 - (int)threadIdx.x);
    unsigned sum = one;
    static_for<0, WAVE_BLOCKS / 8>([&](auto ig) {    // (lanes by immediate numbers: one from a register costs a wait)
        constexpr int g = 8 * decltype(ig)::value;
        if (g >= N) return;
        static_for<0, 8>([&](auto ij) {
            constexpr int j = g + decltype(ij)::value;
            const unsigned add = (unsigned)__builtin_amdgcn_readlane((int)one, j);
            sum += key_at((unsigned)__builtin_amdgcn_readlane((int)word, j), WAVE_BLOCKS - 1 - j) > key ? add : 0u;
        });
    });
    return Ranked{(int)(sum >> 16) - 1, (int)(sum & 0xffffu)};
}

// A set of blocks, a bit each, that is a prefix of the ranked order; its number and its step bits.
struct WaveSet { u64 in; int n, w; };
__device__ __forceinline__ WaveSet prefix_set(const Ranked &r, bool in)
{
    WaveSet s;
    s.in = __ballot(in);
    s.n = __popcll(s.in);
    const u64 last = __ballot(in && r.rank == s.n - 1);
    s.w = s.n ? __builtin_amdgcn_readlane(r.bits, uni(__ffsll((long long)last) - 1)) : 0;
    return s;
}

__device__ __forceinline__ u64 wave_value(u64 v) { return (u64)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), 63) << 32 | (unsigned)__builtin_amdgcn_readlane((int)v, 63); }

template <bool STEP>
__global__ __launch_bounds__(64)
void search_wave_kernel(AllocState *st, AllocHead head, const float *__restrict__ cost, const float *__restrict__ s_up,
                        const float *__restrict__ s_down, const uint8_t *level_in, uint8_t *level_out, sbits_trace *tr, AllocReport *report)
{
    constexpr int PITCH = MAX_CAND | 1;
    __shared__ float table[WAVE_BLOCKS * PITCH];
    __shared__ int bits[MAX_CAND];
    const int lane = (int)threadIdx.x, N = (int)head.N, K = head.K;
    const bool there = lane < N;
    if (lane == 0) {
        st->head = head;
#pragma unroll
        for (int l = 0; l < MAX_CAND; ++l) bits[l] = head.bits[l];   // (a lane each would index the kernel's arguments: scratch)
    }
    __syncthreads();

    // keys as in table_keys and step_keys
    unsigned ku = 0u, kd = 0u, wu = 0u, wd = 0u;
    int lv = head.l0;
    long long used = head.used, k = head.k;
    u64 most = 0ull;                                 // the largest entry of the table
    const float *const row = &table[lane * PITCH];
    if constexpr (STEP) {
        u64 in_use = 0ull;
        lv = there ? (int)level_in[lane] : 0;
        if (there) {
            const int l = min(lv, K - 1);
            const float up = s_up[lane], dn = s_down[lane];
            in_use = (u64)bits[l];
            if (l < K - 1) { ku = some(ord_f32(up)); wu = (unsigned)(bits[l + 1] - bits[l]); }
            if (l > 0) { kd = some(~ord_f32(dn)); wd = (unsigned)(bits[l] - bits[l - 1]); }
        }
        used = (long long)wave_value(wave_reduce<false>(in_use));
    } else {
        if (there) {
            for (int l = 0; l < K; ++l) {
                const float c = cost[(int64_t)lane * K + l];
                if (c > 0.0f) most = max(most, (u64)__float_as_uint(c));
                table[lane * PITCH + l] = c;
            }
        }
        __syncthreads();
        if (there) {
            if (lv < K - 1) {
                wu = (unsigned)(bits[lv + 1] - bits[lv]);
                ku = some(ord_f32((row[lv] - row[lv + 1]) / (float)wu));
            }
            if (lv > 0) {
                wd = (unsigned)(bits[lv] - bits[lv - 1]);
                kd = some(~ord_f32((row[lv - 1] - row[lv]) / (float)wd));
            }
        }
        most = wave_value(wave_reduce<true>(most));
    }

    // The sets of one iteration (see choose_sets): the blocks to raise and, of a swap, those to lower, outside of the set that the
    // raised ones are a prefix of.
    struct Choice { bool expand; WaveSet up, down; };
    auto choose = [&](long long slack) {
        const long long h = k / 2 < 1 ? 1 : k / 2;
        const Ranked up = rank_keys(ku, wu, N);
        Choice c;
        c.up = prefix_set(up, ku >= 0x80000001u && up.rank < k && up.bits <= slack);   // (values above +0)
        c.expand = c.up.n > 0;
        c.down = WaveSet{0ull, 0, 0};
        if (!c.expand) {
            const bool u = ku && up.rank < h;
            const unsigned word = u ? 0u : kd;
            const Ranked down = rank_keys(word, wd, N);
            c.down = prefix_set(down, word && down.rank < h);
            c.up = prefix_set(up, u && up.bits <= slack + c.down.w);
        }
        return c;
    };

    if constexpr (STEP) {
        const Choice c = choose(head.T - used);
        const bool swap = !c.expand && c.up.n && c.down.n;
        const u64 raised = c.expand || swap ? c.up.in : 0ull, lowered = swap ? c.down.in : 0ull;
        if (there) level_out[lane] = (uint8_t)(lv + (int)(raised >> lane & 1ull) - (int)(lowered >> lane & 1ull));
        if (lane == 0 && report) {
            AllocResult r = {};
            r.used = used; r.budget = head.T;
            r.mode = c.expand ? MODE_EXPAND : swap ? MODE_ACCEPT : MODE_NONE;
            r.prop_up = __popcll(raised);
            r.prop_dn = __popcll(lowered);
            r.prop_after = used + (c.expand || swap ? c.up.w - c.down.w : 0);
            r.valid = 1;
            report->result = r;
        }
    } else {
        int shift = 0;
        if (most) {
            const unsigned int b = (unsigned int)most;
            const int x = (int)(b >> 23);
            const int ilog = x ? x - 127 : (31 - __clz((int)(b & 0x7fffffu))) - 149;
            shift = 61 - head.ceil_log2_n - (ilog + 1);
        }
        int iters = 0, expansions = 0, swaps_ok = 0, swaps_rej = 0, status = SBITS_OK;
        bool done = head.done != 0;
        // A block that moves: as in search_kernel, what it cost to leave the old level is, complemented, the key of the way back.
        auto move = [&](int by) {
            if (!by) return;
            const bool up = by > 0;
            lv += by;
            const int from = up ? lv : lv - 1;       // the next step from there
            unsigned word = 0u, step = 0u;
            if (from >= 0 && from < K - 1) {
                step = (unsigned)(bits[from + 1] - bits[from]);
                const unsigned o = ord_f32((row[from] - row[from + 1]) / (float)step);
                word = some(up ? o : ~o);
            }
            const unsigned back = some(~(up ? ku : kd)), wide = up ? wu : wd;
            ku = up ? word : back;
            kd = up ? back : word;
            wu = up ? step : wide;
            wd = up ? wide : step;
        };
        while (!done) {
            const Choice c = choose(head.T - used);
            const int by = (int)(c.up.in >> lane & 1ull) - (int)(c.down.in >> lane & 1ull);
            const long long after = used + c.up.w - c.down.w;
            if (c.expand) {
                move(by);
                if (lane == 0) trace_write(tr, iters, 0, k, c.up.n, 0, c.up.n, 0, used, after, 0);
                used = after;
                ++expansions;
            } else {
                u64 change = 0ull;
                if (by) {
                    const float *entry = row + lv + (by > 0 ? 0 : -1);
                    change = (u64)fx(entry[0] - entry[1], shift);
                    if (by > 0) change = 0ull - change;
                }
                const long long delta = (long long)wave_value(wave_reduce<false>(change));
                if (c.up.n && c.down.n && delta < 0) {
                    move(by);
                    if (lane == 0) trace_write(tr, iters, 1, k, c.up.n, c.down.n, c.up.n, c.down.n, used, after, delta);
                    used = after;
                    ++swaps_ok;
                } else {
                    if (lane == 0) trace_write(tr, iters, 2, k, 0, 0, c.up.n, c.down.n, used, used, delta);
                    k = k / 2;
                    ++swaps_rej;
                }
            }
            ++iters;
            if (k < head.kmin) done = true;
            else if (iters >= head.max_iters) { done = true; status = SBITS_ERR_MAX_ITERS; }
        }
        if (there) level_out[lane] = (uint8_t)lv;
        const u64 total = wave_value(wave_reduce<false>(there ? (u64)fx(row[lv], shift) : 0ull));
        const u64 in_use = wave_value(wave_reduce<false>(there ? (u64)bits[lv] : 0ull));
        if (lane == 0) {
            AllocResult r = {};
            r.used = used; r.k = k; r.budget = head.T; r.shift = shift; r.status = status;
            r.iters = iters; r.expansions = expansions; r.swaps_ok = swaps_ok; r.swaps_rej = swaps_rej;
            r.cost_fixed = (long long)total; r.bits_check = (long long)in_use;
            r.valid = 1;
            report->result = r;
        }
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

static int prep_wgs(int64_t N) { return (int)((N + PREP_THREADS - 1) / PREP_THREADS < PREP_WGS ? (N + PREP_THREADS - 1) / PREP_THREADS : PREP_WGS); }

template <bool STEP>
static void launch_search(hipStream_t sm, unsigned G, const AllocWs &w, int64_t N, const float *cost, const float *s_up,
                          const float *s_down, uint8_t *level, AllocReport *report, int only_if_aborted)
{
    auto *fn = (N + G - 1) / G <= (int64_t)AL_KPT * AL_THREADS ? &search_kernel<STEP, true> : &search_kernel<STEP, false>;
    hipLaunchKernelGGL(fn, dim3(G), dim3(AL_THREADS), 0, sm, w.st, cost, s_up, s_down, level, w.keyU, w.keyD, w.tr, report, prep_wgs(N),
                       SBITS_SPIN_LIMIT, only_if_aborted);
}

static AllocHead start_head(const sbits_plan *plan, double avg_bits)
{
    AllocHead h;
    memset(&h, 0, sizeof h);
    h.N = plan->N;
    h.T = (long long)floor(avg_bits * (double)plan->N);
    h.K = plan->K;
    h.ceil_log2_n = ceil_log2_ll(plan->N);
    h.min_step = 0x7fffffff;
    for (int c = 1; c < plan->K; ++c) if (plan->bits[c] - plan->bits[c - 1] < h.min_step) h.min_step = plan->bits[c] - plan->bits[c - 1];
    for (int c = 0; c < MAX_CAND; ++c) h.bits[c] = c < plan->K ? plan->bits[c] : plan->bits[plan->K - 1];
    return h;
}

// The context's page-locked buffer, ready for the next result.
static int report_buffer(sbits_ctx *ctx, AllocReport **out)
{
    static_assert(sizeof(AllocReport) <= SBITS_PINNED_BYTES, "a result must fit the pinned buffer");
    if (!ctx->pinned) SBITS_HIP(ctx, hipHostMalloc(&ctx->pinned, SBITS_PINNED_BYTES, hipHostMallocDefault));
    *out = static_cast<AllocReport *>(ctx->pinned);
    (*out)->result.valid = 0;
    (*out)->gave_up = 0u;
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
    AllocReport *report;
    const int rc = report_buffer(ctx, &report);
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

    if (N <= WAVE_BLOCKS) {
        hipLaunchKernelGGL(search_wave_kernel<false>, dim3(1), dim3(64), 0, sm, w.st, h0, cost, nullptr, nullptr, nullptr, level, w.tr, report);
        SBITS_HIP(ctx, hipGetLastError());
        return SBITS_OK;
    }
    // The workgroups wait for each other.  Should the device be so full that they never run together, they
    // give up (see give_up) and one workgroup, which waits for nobody, does the search.
    const unsigned G = search_wgs(N, false, ctx->cus);
    hipLaunchKernelGGL(prepare_kernel<false>, dim3(prep_wgs(N)), dim3(PREP_THREADS), 0, sm, w.st, h0, cost, nullptr, nullptr, level, w.keyU, w.keyD);
    launch_search<false>(sm, G, w, N, cost, nullptr, nullptr, level, report, 0);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_SECOND_TRY ? SBITS_OK : stop_if_aborted(ctx, w.st);
}

bool sbits_allocation_failed(const sbits_plan *plan)
{
    const AllocReport *r = static_cast<const AllocReport *>(plan->ctx->pinned);
    return !r->result.valid || r->gave_up;
}

int sbits_repeat_allocate(sbits_plan *plan, const float *cost, uint8_t *level, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    const AllocWs w = alloc_ws(ws, plan->N);
    AllocReport *report;
    const int rc = report_buffer(ctx, &report);
    if (rc) return rc;
    launch_search<false>(ctx->stream, 1, w, plan->N, cost, nullptr, nullptr, level, report, 1);
    SBITS_HIP(ctx, hipGetLastError());
    return SBITS_OK;
}

sbits_alloc_after sbits_after_allocate(const sbits_plan *plan, void *ws)
{
    const AllocWs w = alloc_ws(ws, plan->N);
    return sbits_alloc_after{&w.st->head.aborted, w.keyU};
}

int sbits_finish_allocate(sbits_plan *plan, sbits_stats *host_stats, sbits_trace *host_trace, int64_t trace_cap, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    const AllocResult h = static_cast<const AllocReport *>(ctx->pinned)->result;
    if (sbits_allocation_failed(plan)) return SBITS_ERR_INTERNAL;
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

// One step of Algorithm 2 on caller-supplied estimates.  Workspace as the allocation's.
int sbits_run_propose(sbits_plan *plan, const float *s_up, const float *s_down, const uint8_t *level_in,
                      double avg_bits, int64_t k, uint8_t *level_out, sbits_proposal *host_out, void *ws)
{
    sbits_ctx *ctx = plan->ctx;
    hipStream_t sm = ctx->stream;
    const int64_t N = plan->N;
    const AllocWs w = alloc_ws(ws, N);
    AllocReport *report = nullptr;                                   // (without a host output nothing is waited for)
    const int rc = host_out ? report_buffer(ctx, &report) : SBITS_OK;
    if (rc) return rc;
    AllocHead h = start_head(plan, avg_bits);
    h.k = k;
    // the start state travels as a kernel argument: nothing to keep alive, nothing to wait for
    if (N <= WAVE_BLOCKS) {
        hipLaunchKernelGGL(search_wave_kernel<true>, dim3(1), dim3(64), 0, sm, w.st, h, nullptr, s_up, s_down, level_in, level_out, nullptr, report);
    } else {
        const unsigned G = search_wgs(N, true, ctx->cus);
        uint8_t *const lv = const_cast<uint8_t *>(level_in);             // (only read by the step)
        hipLaunchKernelGGL(prepare_kernel<true>, dim3(prep_wgs(N)), dim3(PREP_THREADS), 0, sm, w.st, h, nullptr, s_up, s_down, lv, w.keyU, w.keyD);
        launch_search<true>(sm, G, w, N, nullptr, s_up, s_down, lv, report, 0);
        if (G > 1 && SBITS_SECOND_TRY) launch_search<true>(sm, 1, w, N, nullptr, s_up, s_down, lv, report, 1);   // returns at once unless the first gave up
        const unsigned grid = (unsigned)((N + 255) / 256 < 1024 ? (N + 255) / 256 : 1024);
        hipLaunchKernelGGL(step_apply_kernel, dim3(grid), dim3(256), 0, sm, (const AllocState *)w.st,
                           (const u64 *)w.keyU, (const u64 *)w.keyD, level_in, level_out);
    }
    SBITS_HIP(ctx, hipGetLastError());
    if (host_out) {
        SBITS_HIP(ctx, hipStreamSynchronize(sm));
        const AllocResult r = report->result;            // (of the second launch, if the first gave up)
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
