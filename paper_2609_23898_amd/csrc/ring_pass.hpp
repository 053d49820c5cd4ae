// The one-pass all-reduce: its launch parameters and rules.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "cerar_internal.hpp"

namespace cerar {

// One independent all-reduce (a bucket): its buffers and geometry.
struct PassInst {
    const float *grads;
    float *out, *work, *pool;      // work == nullptr: only `out` is written
    size_t d, p, pool_stride;
    unsigned blk0;                 // first of its blocks (or runs) in the call's numbering
};

constexpr int kPassInst = 32;

struct PassParams {
    size_t ld_g, ld_o, ld_w;
    const float *efrag, *dfrag;    // N x MT x KSe x 64 and N x MT x KSd x 64
    const uint16_t *esplit, *dsplit;   // the split operands, N x 2 KC tiles
    int N, c, KSe, KSd, n;
    unsigned nblk;                 // blocks (split kernels: runs of blocks) of all instances
    unsigned run;                  // split kernels: half-blocks per workgroup
    int coefs;                     // split kernels: SplitCoefs of the plan
    int ragged;                    // some row of grads or out does not start on a 128-byte line
    PassInst in[kPassInst];
};
static_assert(sizeof(PassParams) <= 4096, "kernel arguments");

constexpr size_t kPassLds = 160 * 1024;

// LDS floats of one worker's rows: K rows of P positions, and an offset that
// keeps the workers' rows of one position in different banks.
__host__ __device__ inline int pass_region(int N, int K, int P) { return K * P + ((64 / N) & ~3); }
inline size_t pass_lds(int N, int c, int V) { return (size_t)N * pass_region(N, c + N - 1, 16 * V) * sizeof(float); }

// Positions of one workgroup's block for this plan, or 0 where the one-pass
// kernel does not take it.
int pass_positions(int N, int c);
// The workgroups per CU of the plan's own kernels on the current device, looked
// up once, so that a launch, which may be under stream capture, only launches.
hipError_t prepare_passes(int N, int c, PassSize *out);
// One launch; cus: compute units of the current device.
void launch_ring_pass(const PassParams &a, int cus, const PassSize &size, hipStream_t s);

// The rounds alone, where the call does not go in one pass: reads the encoded chunks in `work`
// (grads and out unused); 0 where N is too large for it.
int rounds_positions(int N);
void launch_rounds_pass(const PassParams &a, int cus, const PassSize &size, hipStream_t s);

// Encode and decode on split operands (plans with KC = split_chunks > 0): the
// half-blocks (32 positions) per workgroup for this many in all, and the
// launches, of N nblk workgroups.
unsigned split_run(int N, int KC, int cus, size_t half_blocks);
void launch_encode_split(const PassParams &a, int KC, hipStream_t s);
void launch_decode_split(const PassParams &a, int KC, hipStream_t s);

}  // namespace cerar
