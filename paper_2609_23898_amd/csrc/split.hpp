// The contraction on bf16 MFMAs at fp32 accuracy: device helpers.
//
// Every fp32 operand x is split exactly into three bf16 terms, x = h + m + l:
// h is x rounded to bf16 (round to nearest even), m the remainder rounded to
// bf16, l the rest, which bf16 holds exactly (8 significant bits).  Of the
// nine products of two split operands the six with h h, h m, m h, h l, m m,
// l h are kept; each is exact in fp32, and since |m| <= 2^-8 |x| (1 + 2^-8)
// and |l| <= 2^-16 |x|, the dropped m l, l m and l l sum to less than 2^-23
// |a||b|, two units of fp32 rounding, so a product is fp32-accurate (the
// six-product scheme of Henry, Tang and Heinecke, "Leveraging the bfloat16
// artificial intelligence datatype for higher-precision computations", ARITH
// 2019).  The 16x16x32 bf16 MFMA does 32 K-steps in half the cycles the fp32
// one takes for 4, so the six products cost 3/8 of the fp32 MFMA time, and
// other waves' vector instructions run beside it, which the fp32 MFMA excludes
// (measured: 4 MFMAs and 32 FMAs of two waves take 130 + 180 -> 313 cycles with
// fp32, 80 + 175 -> 210 with bf16).
//
// The terms hold an entry exactly from 2^-110 (below that the last one falls
// under bf16's smallest subnormal, 2^-133) up to 2^127 (beyond, the first could
// round to infinity).  A half-block of 32 positions with another entry in it
// (SplitRange) loses no digit either:
//  - The encode, with small entries and none of 2^40 or more, scales all of them
//    by 2^40 (fp32's smallest subnormal becomes 2^-109) and its chunks back.
//    Plans with coefficients of 2^40 or more, whose sums could overflow so, do
//    not scale.
//  - Any other such half-block, and every one of a plan that has a coefficient
//    like that, is contracted on fp32 MFMAs (tiles_f32).  In the decode, whose
//    rows are sums over workers and chunks, small ones are that rare.
// The test costs one vector instruction per entry beside five and a half of the
// split (us, without and with: encode N = 16, c = 128, d = 1e8 2759 and 2759, N = 20,
// c = 40, d = 20M 743 and 731, N = 3, c = 100, d = 1e8 623 and 638; single call N = 16, c =
// 64, d = 40M 2359 and 2415, N = 12, c = 48 2374 and 2250); zeros take a second look.
// Entries of 1e-36, d = 20M: one in a thousand N = 16, c = 64 encode 530 us as without,
// 1022 on fp32 MFMAs; all of them, decode 3.3 ms against 0.6.
#pragma once

#include <hip/hip_runtime.h>

#include "cerar_internal.hpp"
#include "device_util.hpp"
#include "rows.hpp"

namespace cerar {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

template <class V>
struct Split3 { V h, m, l; };

// What stands in for a reduction row that the plan does not have; its
// coefficients are zero.  No zero, which SplitRange would look at twice.
constexpr v2f kNoRow = {1.f, 1.f};

// acc += A B for split A and B with the six kept products, the small ones first.
__device__ inline v4f mma_split32(const Split3<v8bf> &a, const Split3<v8bf> &b, v4f acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b.m, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.m, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, acc, 0, 0, 0);
}
__device__ inline v4s as_v4s(v4bf v) { return __builtin_bit_cast(v4s, v); }
__device__ inline v4f mma_split16(const Split3<v4bf> &a, const Split3<v4bf> &b, v4f acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.l), as_v4s(b.h), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.m), as_v4s(b.m), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.h), as_v4s(b.l), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.m), as_v4s(b.h), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.h), as_v4s(b.m), acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a.h), as_v4s(b.h), acc, 0, 0, 0);
}

// One tile's A operands (the layout of split_tile_encode / split_tile_decode),
// in LDS or global memory.
__device__ inline Split3<v8bf> tile_a32(const __bf16 *tile, int kc, uint32_t lane) {
    const __bf16 *b = tile + (size_t)kc * 3 * 64 * 8 + lane * 8;
    return {*reinterpret_cast<const v8bf *>(b), *reinterpret_cast<const v8bf *>(b + 64 * 8),
            *reinterpret_cast<const v8bf *>(b + 2 * 64 * 8)};
}
__device__ inline Split3<v4bf> tile_a16(const __bf16 *tile, int KC, uint32_t lane) {
    const __bf16 *b = tile + (size_t)KC * 3 * 64 * 8 + lane * 4;
    return {*reinterpret_cast<const v4bf *>(b), *reinterpret_cast<const v4bf *>(b + 64 * 4),
            *reinterpret_cast<const v4bf *>(b + 2 * 64 * 4)};
}

// Two values at once (one packed conversion per term); returns the three
// terms as packed bf16 pairs.
__device__ inline void split3_pair(v2f x, uint32_t &h, uint32_t &m, uint32_t &l) {
    const v2bf xh = __builtin_convertvector(x, v2bf);
    const v2f r = x - __builtin_convertvector(xh, v2f);        // exact
    const v2bf xm = __builtin_convertvector(r, v2bf);
    const v2bf xl = __builtin_convertvector(r - __builtin_convertvector(xm, v2f), v2bf);   // exact
    h = __builtin_bit_cast(uint32_t, xh);
    m = __builtin_bit_cast(uint32_t, xm);
    l = __builtin_bit_cast(uint32_t, xl);
}
// Eight (four) K-steps of one position: x(s) is the value of step s.
template <class X>
__device__ inline Split3<v8bf> split8(X x) {
    v4u h, m, l;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t th, tm, tl;
        split3_pair(v2f{x(2 * w), x(2 * w + 1)}, th, tm, tl);
        h[w] = th;
        m[w] = tm;
        l[w] = tl;
    }
    return {__builtin_bit_cast(v8bf, h), __builtin_bit_cast(v8bf, m), __builtin_bit_cast(v8bf, l)};
}
template <class X>
__device__ inline Split3<v4bf> split4(X x) {
    v2u h, m, l;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        uint32_t th, tm, tl;
        split3_pair(v2f{x(2 * w), x(2 * w + 1)}, th, tm, tl);
        h[w] = th;
        m[w] = tm;
        l[w] = tl;
    }
    return {__builtin_bit_cast(v4bf, h), __builtin_bit_cast(v4bf, m), __builtin_bit_cast(v4bf, l)};
}

// How a half-block is contracted.
enum Contract { kUsual, kScaled, kFp32 };
constexpr float kScale = 0x1p40f;

// Whether the wave has met an entry that its three terms do not hold exactly.
// (A NaN makes NaNs of its position either way.)
struct SplitRange {
    float lo = 1.f, hi = 1.f;                             // least and largest magnitude
    __device__ void add(v2f x) {                          // as asm, or the compiler quiets each operand first
        asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(lo) : "v"(x[0]), "v"(x[1]));
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(hi) : "v"(x[0]), "v"(x[1]));
    }
    // coefs: see PassParams; each(f) calls f on every entry again, to tell zeros
    // from small ones
    template <class Each>
    __device__ Contract contract(int coefs, Each each) const {
        if (coefs == kCoefsFp32) return kFp32;
        if (__builtin_amdgcn_ballot_w64(lo < 0x1p-110f || hi >= 0x1p127f) == 0) return kUsual;
        if (__builtin_amdgcn_ballot_w64(hi >= 0x1p127f) != 0) return kFp32;
        uint32_t least = 0xffffffffu;                     // of 2 bits - 1: a zero wraps to the largest
        each([&](v2f x) { least = min(least, min((__float_as_uint(x[0]) << 1) - 1, (__float_as_uint(x[1]) << 1) - 1)); });
        if (__builtin_amdgcn_ballot_w64(least < 2u * (17u << 23) - 1) == 0) return kUsual;
        return coefs == kCoefsUsual && __builtin_amdgcn_ballot_w64(hi >= 0x1p40f) == 0 ? kScaled : kFp32;
    }
};

// The contraction of a rare half-block on fp32 MFMAs: the first `tiles` of TILES
// tiles at W positions a lane.  frag has their fp32 coefficients, KS K-steps of
// 64 lanes a tile; row(k, t) gives reduction row k at the lane's position t.
// Where it costs the usual path registers it is called out of line (the one-pass
// encode: N = 9, c = 64, d = 40M 1.80 ms so, 1.90 inline); the step encode is
// faster with its own inline (N = 12, c = 48, d = 40M: 844 against 890 us).
#define CERAR_RARE __device__ __attribute__((noinline))
template <int TILES, int W, class Row>
__device__ inline void tiles_f32(v4f (&acc)[TILES][W], int tiles, const float *frag, int KS, int lane, Row row) {
#pragma unroll
    for (int mt = 0; mt < TILES; ++mt)
#pragma unroll
        for (int t = 0; t < W; ++t) acc[mt][t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int ks = 0; ks < KS; ++ks) {
        float y[W];
#pragma unroll
        for (int t = 0; t < W; ++t) y[t] = row(4 * ks + (lane >> 4), t);
#pragma unroll
        for (int mt = 0; mt < TILES; ++mt)
            if (mt < tiles) {
                const float coef = gload1(frag + (size_t)(mt * KS + ks) * 64 + lane);
#pragma unroll
                for (int t = 0; t < W; ++t) acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(coef, y[t], acc[mt][t], 0, 0, 0);
            }
    }
}

// The same for the encode, one tile with the K-steps in the order of its
// registers: x(kc, s, t) gives row 32 kc + 8 g + s of lane group g.  UNROLL: all
// 8 KC of them where x is in registers, else 1.
template <int KC, int UNROLL, class X>
__device__ inline void tile_f32(v4f (&acc)[2], const float *frag, int KS, int lane0, X x) {
    const uint32_t lane = opaque((uint32_t)lane0), ks0 = 2 * (lane >> 4);
    const float *a = frag + ks0 * 64 + (lane & 15);
    acc[0] = acc[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll UNROLL
    for (int u = 0; u < 8 * KC; ++u) {
        const int kc = u / 8, s = u % 8, ks = 8 * kc + s / 4;
        const float coef = (int)ks0 + ks < KS ? gload1(a + ks * 64 + s % 4 * 16) : 0.f;
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(coef, x(kc, s, 0), acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(coef, x(kc, s, 1), acc[1], 0, 0, 0);
    }
}

// The end of a rare half-block's path, where loads for the next one are under
// way: waits for all of them.  Where it meets the usual path the compiler would
// otherwise take the fewer stores issued here after those loads for both, and
// wait for the usual path's stores as well.
__device__ inline void wait_all() { __builtin_amdgcn_s_waitcnt(0); }

}  // namespace
}  // namespace cerar
