// Device helpers shared by the kernels' translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cerar {
namespace {

// Hides a value's loop invariance from the compiler (it emits no
// instruction), so that base + offset is not hoisted into one live 64-bit
// pointer per row across a block loop.
__device__ inline uint32_t opaque(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The same for a wave-uniform value (kept in scalar registers).
__device__ inline size_t opaque_s(size_t x) {
    asm volatile("" : "+s"(x));
    return x;
}

// The next message of a round N <= k < c, x = recv - delta_j + delta_{k+1},
// rounded to fp32 once: the three fp32 terms are combined in fp64 (the
// difference of two fp32 values is exact there unless their exponents are
// more than 29 apart), so a message carries one rounding per round instead
// of two.  A message keeps the rounding error of every earlier round (the
// returning own term cancels, its rounding does not), and the decode
// amplifies those errors by up to kappa_2(M_i), so this is the round's
// share of the final error.
__device__ inline float combine3(float recv, float sub, float add) {
    return (float)(((double)recv - (double)sub) + (double)add);
}

// Index of the last instance whose first workgroup is at or before `block`.
template <class Inst>
__device__ inline int instance_of(const Inst *in, int n, unsigned block) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (in[mid].wg0 <= block) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace
}  // namespace cerar
