// Accesses to rows of floats in global memory, shared by the kernels that take
// rows of any alignment.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.hpp"

namespace cerar {
namespace {

// V floats of one row; rows may start at any float, so the accesses claim
// four-byte alignment only.
template <int V>
struct Vec {
    typedef float T __attribute__((ext_vector_type(V)));
    typedef float U __attribute__((ext_vector_type(V), aligned(4)));
};
template <int V>
__device__ inline typename Vec<V>::T gload(const float *ubase, uint32_t lane_bytes) {
    typedef __attribute__((address_space(1))) const typename Vec<V>::U GU;
    typedef __attribute__((address_space(1))) const char GC;
    return *(GU *)((GC *)ubase + lane_bytes);
}
template <int V>
__device__ inline typename Vec<V>::T gload_nt(const float *ptr) {
    typedef __attribute__((address_space(1))) const typename Vec<V>::U GU;
    return __builtin_nontemporal_load((GU *)ptr);
}
template <int V>
__device__ inline void gstore(float *ubase, uint32_t lane_bytes, typename Vec<V>::T v) {
    typedef __attribute__((address_space(1))) typename Vec<V>::U GU;
    typedef __attribute__((address_space(1))) char GC;
    __builtin_nontemporal_store((typename Vec<V>::U)v, (GU *)((GC *)ubase + lane_bytes));
}
template <int V>
__device__ inline void gstore_cached(float *ubase, uint32_t lane_bytes, typename Vec<V>::T v) {
    typedef __attribute__((address_space(1))) typename Vec<V>::U GU;
    typedef __attribute__((address_space(1))) char GC;
    *(GU *)((GC *)ubase + lane_bytes) = v;
}
__device__ inline float gload1(const float *ptr) { return *(__attribute__((address_space(1))) const float *)ptr; }
__device__ inline void gstore1(float *ptr, float v) { *(__attribute__((address_space(1))) float *)ptr = v; }

// ptr + floats for a wave-uniform ptr, kept from being rewritten as base +
// row x p: one live scalar pointer that steps from row to row instead of one
// per row.
template <class T>
__device__ inline T *step(T *ptr, size_t floats) {
    const size_t v = reinterpret_cast<size_t>(ptr + floats);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<T *>(opaque_s((size_t)hi << 32 | lo));
}

// Rows up to this length have the byte offsets of 13 rows in 32 bits (a
// scalar base and a 32-bit lane offset); longer ones are addressed in 64 bits.
constexpr size_t kNarrow = (size_t)1 << 26;

}  // namespace
}  // namespace cerar
