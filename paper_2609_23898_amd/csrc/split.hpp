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
// fp32, 80 + 175 -> 210 with bf16).  Values must lie in bf16's range (|x| <
// 3.39e38); terms below fp32's normal range lose their low bits.
#pragma once

#include <hip/hip_runtime.h>

#include "cerar_internal.hpp"
#include "device_util.hpp"

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

}  // namespace
}  // namespace cerar
