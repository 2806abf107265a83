// Arithmetic core of the packing stage: re-quantization of one block row at the block's chosen
// bitwidth (paper Sec. 5 "Implementation": asymmetric min-max round-to-nearest grid, group =
// one block row) and the little-endian bit string of a lane's 8 codes.  Shared by the kernel
// that reads reordered weights and by the one that reorders on the fly.
#pragma once

#include "sbits_device.hpp"

namespace sbits {

// bitwidth, qmax and the finite-quotient threshold of candidate `lv` (c == 0: a pruned block)
struct LevelConsts {
    int c;
    float qf, th;
    unsigned int qmax;
    unsigned int keep;       // all ones, or 0 for a pruned block: ANDed onto the bits of the group minimum
};
// (one AND per row; a compare-and-select on c here costs the packing kernel 5 %)
__device__ __forceinline__ float origin_of(const LevelConsts &k, float lo)
{
    return __uint_as_float(__float_as_uint(lo) & k.keep);
}
__device__ __forceinline__ LevelConsts level_consts(const GridConsts &gc, int lv)
{
    LevelConsts k;
    k.c = gc.bits[0]; k.qf = gc.qmaxf[0]; k.th = gc.thr[0];
#pragma unroll
    for (int cc = 1; cc < MAX_CAND; ++cc)
        if (lv == cc) { k.c = gc.bits[cc]; k.qf = gc.qmaxf[cc]; k.th = gc.thr[cc]; }
    k.qmax = (unsigned int)k.qf;
    k.keep = k.c ? 0xffffffffu : 0u;
    return k;
}

// One row of one lane group: raw = the lane's 8 bf16 weights.  Returns the lane's 8 codes,
// code e in bits [e*c, (e+1)*c); scl / mn are the row's scale and minimum (same in all lanes
// of the group).  Even lanes divide qmax / R, odd lanes R / qmax.
template <int LPG>
__device__ __forceinline__ unsigned long long quant_pack_row(const uint4 &raw, const LevelConsts &k, bool odd,
                                                             float &scl, float &mn)
{
    float w[8];
    unpack8(raw, w);
    mn = fminf(fminf(fminf(w[0], w[1]), fminf(w[2], w[3])), fminf(fminf(w[4], w[5]), fminf(w[6], w[7])));
    float mx = fmaxf(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3])), fmaxf(fmaxf(w[4], w[5]), fmaxf(w[6], w[7])));
    mn = group_allreduce<LPG>(mn, OpMin{});
    mx = group_allreduce<LPG>(mx, OpMax{});
    const float R = mx - mn;
    mn = origin_of(k, mn);                           // pruned block: origin 0 (both quotients are 0 by its threshold)
    float inv;
    if (LPG >= 2) {
        float v = (odd ? R : k.qf) / (odd ? k.qf : R);
        if (R < k.th) v = 0.0f;
        inv = group_bcast<LPG, 0>(v);
        scl = group_bcast<LPG, 1 % LPG>(v);
    } else {
        inv = k.qf / R; scl = R / k.qf;
        if (R < k.th) { inv = 0.0f; scl = 0.0f; }
    }
    // q = rint(y) for 0 <= y < 2^22 sits in the low mantissa bits of y + 1.5 * 2^23 (round to
    // nearest even, as rintf); y <= qmax * (1 + 2^-22) here, so rint(y) <= qmax and the mask only
    // guards the neighbours' bits against non-finite input.  4 codes fit in 32 bits (c <= 8).
    uint32_t half[2];
#pragma unroll
    for (int hq = 0; hq < 2; ++hq) {
        uint32_t acc = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float y = (w[4 * hq + e] - mn) * inv;
            const uint32_t q = __float_as_uint(y + 12582912.0f) & k.qmax;
            acc |= q << (e * k.c);
        }
        half[hq] = acc;
    }
    const unsigned long long word = (unsigned long long)half[0] | ((unsigned long long)half[1] << (4 * k.c));
    return word;
}

// RS rows of one lane group at once (w[rs] = the lane's 8 weights of row rs), LPG >= 2 * RS: the
// 2 * RS grid quotients are spread over the lanes of the group (lane 2*rs: qmax / R of row rs,
// lane 2*rs + 1: R / qmax), so the rows share ONE division sequence instead of paying one each.
// Same results as quant_pack_row row by row, the codes in two halves: code 4 h + e in bits [e*c, (e+1)*c) of half[.][h].
template <int LPG, int RS>
__device__ __forceinline__ void quant_pack_rows(const float (&w)[RS][8], const LevelConsts &k, int lig,
                                                uint32_t (&half)[RS][2], float (&scl)[RS], float (&mn)[RS])
{
    static_assert(LPG >= 2 * RS, "one lane per quotient");
    float R[RS];
#pragma unroll
    for (int rs = 0; rs < RS; ++rs) {
        float lo = fminf(fminf(fminf(w[rs][0], w[rs][1]), fminf(w[rs][2], w[rs][3])),
                         fminf(fminf(w[rs][4], w[rs][5]), fminf(w[rs][6], w[rs][7])));
        float hi = fmaxf(fmaxf(fmaxf(w[rs][0], w[rs][1]), fmaxf(w[rs][2], w[rs][3])),
                         fmaxf(fmaxf(w[rs][4], w[rs][5]), fmaxf(w[rs][6], w[rs][7])));
        lo = group_allreduce<LPG>(lo, OpMin{});
        hi = group_allreduce<LPG>(hi, OpMax{});
        mn[rs] = origin_of(k, lo);                   // pruned block: origin 0 (both quotients are 0 by its threshold)
        R[rs] = hi - lo;
    }
    const int qi = lig & (2 * RS - 1);               // lanes beyond 2*RS repeat a quotient; nobody reads theirs
    float Rsel = R[0];
#pragma unroll
    for (int rs = 1; rs < RS; ++rs)
        if ((qi >> 1) == rs) Rsel = R[rs];
    const bool odd = (qi & 1) != 0;
    float v = (odd ? Rsel : k.qf) / (odd ? k.qf : Rsel);        // IEEE correctly rounded
    if (Rsel < k.th) v = 0.0f;
    static_for<0, RS>([&](auto irs) {
        constexpr int rs = decltype(irs)::value;
        const float inv = group_bcast<LPG, 2 * rs>(v);
        scl[rs] = group_bcast<LPG, 2 * rs + 1>(v);
#pragma unroll
        for (int hq = 0; hq < 2; ++hq) {
            uint32_t acc = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float y = (w[rs][4 * hq + e] - mn[rs]) * inv;
                const uint32_t q = __float_as_uint(y + 12582912.0f) & k.qmax;   // see quant_pack_row
                acc |= q << (e * k.c);
            }
            half[rs][hq] = acc;
        }
    });
}

// Transposes a 4 x 4 matrix over the lanes of a quad: on return a[i] is what lane i of the quad held in a[own lane].
__device__ __forceinline__ void quad_transpose(uint32_t (&a)[4], int lane)
{
    auto swap = [&](uint32_t &lo, uint32_t &hi, bool odd, auto ctrl) {
        const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(odd ? lo : hi), decltype(ctrl)::value, 0xf, 0xf, true);
        lo = odd ? got : lo;
        hi = odd ? hi : got;
    };
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
    swap(a[0], a[1], b0, std::integral_constant<int, DPP_XOR1>{});
    swap(a[2], a[3], b0, std::integral_constant<int, DPP_XOR1>{});
    swap(a[0], a[2], b1, std::integral_constant<int, DPP_XOR2>{});
    swap(a[1], a[3], b1, std::integral_constant<int, DPP_XOR2>{});
}

// Codes of four consecutive rows of a block (lo / hi: the low and high words of the 8 c bits that this lane has of each row) to
// the stream.  Four lanes have 32 codes of a row, which are c whole words: after a transposition lane j of a quad has
// those of row j, puts them together and stores them at once; the rows' bytes are consecutive, so a lane group's stores cover one
// run.  dst: the first row's bytes.  WIDE: c may be more than 4 (else hi is not used).
// (Collecting a group's bytes in LDS took two or three atomic ORs a lane and row, which with the column gather filled the LDS
// pipe: two 8B-shaped layers in 64-column blocks at 1 to 8 bits 303 us, 269 this way; the 8192-column rows of the 70B-shaped layer 370,
// with two row buffers besides 330; the 14336-column rows of the 8B-shaped model 1137, 1076; its 4096-column rows, whose stream of weights is the
// slower part, 2.7 ms both.)
// The words leave with nontemporal stores: isolated writes that linger in the caches cost the stream of weights more than their bytes
// (sixteen 8B-shaped layers, 128-column blocks: 1951 -> 1711 us, four at 1 to 8 bits 515 -> 472, the 70B-shaped layer 526 -> 501).  Scale and
// zero, 16 bytes a block at a time, are put together by the L2: nontemporal they cost 20 %.  So are codes of 7 bits and, in 64-column
// blocks, of 3, 5 and 6, whose stores end inside of lines (32768 x 4096 at 7 bits, 128 columns 90 us, nontemporal 94, 64 columns 96 and 121, 5
// bits there 91 and 97; 3 bits and mixed widths within 2 %).
template <int LPG, bool WIDE>
__device__ __forceinline__ void store_codes4(uint8_t *dst, int c, uint32_t (&lo)[4], uint32_t (&hi)[4], int lig)
{
    quad_transpose(lo, lig);
    if constexpr (WIDE) quad_transpose(hi, lig);
    typedef __attribute__((address_space(1))) uint32_t *gp;
    typedef unsigned int u2_t __attribute__((ext_vector_type(2), aligned(4)));
    typedef unsigned int u3_t __attribute__((ext_vector_type(3), aligned(4)));
    typedef unsigned int u4_t __attribute__((ext_vector_type(4), aligned(4)));
    const gp p = (gp)(dst + (lig & 3) * (LPG * c) + (lig >> 2) * 4 * c);
    constexpr std::true_type nt{};
    constexpr std::false_type plain{};
    constexpr std::integral_constant<bool, (LPG >= 16)> gaps{};
    auto put1 = [&](auto past, int at, uint32_t a) {
        __attribute__((address_space(1))) uint32_t *q = (__attribute__((address_space(1))) uint32_t *)(p + at);
        if constexpr (decltype(past)::value) __builtin_nontemporal_store(a, q);
        else *q = a;
    };
    auto put2 = [&](auto past, int at, uint32_t a, uint32_t b) {
        __attribute__((address_space(1))) u2_t *q = (__attribute__((address_space(1))) u2_t *)(p + at);
        if constexpr (decltype(past)::value) __builtin_nontemporal_store(u2_t{a, b}, q);
        else *q = u2_t{a, b};
    };
    auto put3 = [&](auto past, int at, uint32_t a, uint32_t b, uint32_t d) {
        __attribute__((address_space(1))) u3_t *q = (__attribute__((address_space(1))) u3_t *)(p + at);
        if constexpr (decltype(past)::value) __builtin_nontemporal_store(u3_t{a, b, d}, q);
        else *q = u3_t{a, b, d};
    };
    auto put4 = [&](auto past, int at, uint32_t a, uint32_t b, uint32_t d, uint32_t e) {
        __attribute__((address_space(1))) u4_t *q = (__attribute__((address_space(1))) u4_t *)(p + at);
        if constexpr (decltype(past)::value) __builtin_nontemporal_store(u4_t{a, b, d, e}, q);
        else *q = u4_t{a, b, d, e};
    };
    switch (c) {                                     // (a wave has up to eight blocks, of different bitwidths)
    case 0: break;
    case 1: put1(nt, 0, lo[0] | lo[1] << 8 | lo[2] << 16 | lo[3] << 24); break;
    case 2: put2(nt, 0, lo[0] | lo[1] << 16, lo[2] | lo[3] << 16); break;
    case 3: put3(gaps, 0, lo[0] | lo[1] << 24, lo[1] >> 8 | lo[2] << 16, lo[2] >> 16 | lo[3] << 8); break;
    case 4: put4(nt, 0, lo[0], lo[1], lo[2], lo[3]); break;
    default:
        if constexpr (WIDE) switch (c) {
        case 5:
            put4(gaps, 0, lo[0], hi[0] | lo[1] << 8, lo[1] >> 24 | hi[1] << 8 | lo[2] << 16, lo[2] >> 16 | hi[2] << 16 | lo[3] << 24);
            put1(gaps, 4, lo[3] >> 8 | hi[3] << 24);
            break;
        case 6:
            put4(gaps, 0, lo[0], hi[0] | lo[1] << 16, lo[1] >> 16 | hi[1] << 16, lo[2]);
            put2(gaps, 4, hi[2] | lo[3] << 16, lo[3] >> 16 | hi[3] << 16);
            break;
        case 7:
            put4(plain, 0, lo[0], hi[0] | lo[1] << 24, lo[1] >> 8 | hi[1] << 24, hi[1] >> 8 | lo[2] << 16);
            put3(plain, 4, lo[2] >> 16 | hi[2] << 16, hi[2] >> 16 | lo[3] << 8, lo[3] >> 24 | hi[3] << 8);
            break;
        default:
            put4(nt, 0, lo[0], hi[0], lo[1], hi[1]);
            put4(nt, 4, lo[2], hi[2], lo[3], hi[3]);
            break;
        }
    }
}

// the lane's c bytes (c <= 8) of a row's code stream, low byte first; written one by one with
// fixed shifts (a counted loop here gets vectorised into something far more expensive)
template <class BytePtr>
__device__ __forceinline__ void store_code_bytes(BytePtr mine, unsigned long long word, int c)
{
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t < c) mine[t] = (unsigned char)(word >> (8 * t));
}

}  // namespace sbits
