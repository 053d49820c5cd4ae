// HIP kernels for gfx950 and the device-side C ABI of libcerar.
//
//  k_encode  (K1)  delta_{i,j} = sum_l U_i[l][j] chunk_l(g_i), all workers,
//                  as fp32 MFMA 16x16x4 tiles: delta^T = U^T G^T, positions
//                  on the MFMA N axis, coefficients (A operand) from LDS (plans
//                  that contract on split operands: split.hip).
//  k_round   (K2/K3) one ring round for all workers: next message =
//                  received (- returning own term) (+ next own term).
//  k_decode  (K4)  g_hat_i = Y_i R_i, the same MFMA tiling over the L+1
//                  stored observations, gathered through the slot table
//                  (split.hip as above).
//  k_norms   (K5)  per-worker squared error against S = sum_w g_w, fp64,
//                  and on sampled positions against given reference values.
//  k_copy          plain streaming copy (bandwidth reference).
//
// The whole-ring entry points go in one pass (ring_pass.hip) where the plan
// and the buffers allow it; the kernels here are the step calls, and the
// contractions of the whole ring otherwise (its rounds too beyond N = 16).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "cerar_internal.hpp"
#include "device_util.hpp"
#include "ring_pass.hpp"

namespace cerar {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
// Loads through a pointer the compiler cannot place (one read from LDS, as
// the decode's row table) would be flat loads, which count against the LDS
// wait counter too and so serialise the table reads with the data loads.
// Every buffer here is global memory: say so.
// Rows may start at any float: vector accesses claim four-byte alignment only,
// which the hardware takes at full width.  One float at a time, odd d at N = 8,
// c = 64 (d = 60000001) ran a step-call ring in 4.06 ms against 3.48 so, the
// encode 1416 us against 920; an odd work pointer at d = 64000000 6.00 ms against 3.60.
typedef float v4u4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float v2u4 __attribute__((ext_vector_type(2), aligned(4)));
typedef __attribute__((address_space(1))) const v4u4 global_cv4f;
typedef __attribute__((address_space(1))) const float global_cf;
__device__ inline v4f nt_load_g(const float *ptr) { return __builtin_nontemporal_load((global_cv4f *)(ptr)); }
__device__ inline v4f load_g(const float *ptr) { return *(global_cv4f *)(ptr); }
__device__ inline float load1_g(const float *ptr) { return *(global_cf *)(ptr); }

constexpr int kThreads = 256;                  // 4 wavefronts of 64
constexpr int kWaves = kThreads / 64;
constexpr size_t kLdsBudget = 80 * 1024;       // bytes of LDS a workgroup may use (two per 160 KiB CU)

// Address of a p-float slot (see RingTables): the workers' own chunks in
// `work`, or the per-worker message pool in the workspace.
struct SlotBase {
    float *work;
    size_t ld_work;
    size_t p;
    float *pool;
    size_t pool_stride;
    int Nc;
    int c;
    __device__ __host__ float *ptr(int s) const {
        return s < Nc ? work + (size_t)(s / c) * ld_work + (size_t)(s % c) * p
                      : pool + (size_t)(s - Nc) * pool_stride;
    }
};

// ---- position-tile I/O -------------------------------------------------------
// A wave covers 64 consecutive positions e0..e0+63 of one p-float row: lane
// (krow, col) holds positions e0 + 4 col + t, t = 0..3, and MFMA number t works
// on component t.  Entries at or beyond `limit` (flat index row_off + pos) read
// as zero.

__device__ inline v4f load_tile(const float *__restrict__ row, size_t row_off, size_t e0, int col,
                                size_t p, size_t limit) {
    v4f v = {0.f, 0.f, 0.f, 0.f};
    const size_t pos = e0 + 4 * (size_t)col;
    if (pos < p) {
        const size_t flat = row_off + pos;
        if (flat + 3 < limit) {
            v = load_g(row + pos);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (flat + t < limit) v[t] = load1_g(row + pos + t);
        }
    }
    return v;
}

__device__ inline void store_tile(float *__restrict__ row, size_t row_off, size_t e0, int col, size_t p,
                                  size_t limit, v4f v) {
    const size_t pos = e0 + 4 * (size_t)col;
    if (pos < p) {
        const size_t flat = row_off + pos;
        if (flat + 3 < limit) {
            *reinterpret_cast<v4u4 *>(row + pos) = v;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (flat + t < limit) row[pos + t] = v[t];
        }
    }
}

// ---- MFMA operand helpers ------------------------------------------------------
// A fragments (coefficients) are either held in registers for up to four
// M-tiles, or staged in LDS so that one ds_read_b128 fetches four K-steps.
// Interior 64-position blocks (the uniform common case) use unmasked
// non-temporal 16-byte loads and stores; tail blocks take the masked path.

constexpr int kMaxRegTiles = 4;
constexpr int kMaxDecodeKS = 48;   // K = c + N - 1 <= 191 observations

__device__ inline v4f nt_load(const float *ptr) { return __builtin_nontemporal_load(reinterpret_cast<const v4u4 *>(ptr)); }
__device__ inline void nt_store(float *ptr, v4f v) { __builtin_nontemporal_store((v4u4)v, reinterpret_cast<v4u4 *>(ptr)); }

// Wave-uniform base pointer plus a 32-bit per-lane byte offset: the form of a
// global access with a scalar base register, which keeps one VGPR of address
// per lane instead of a 64-bit pointer per row.  opaque() hides the offset's
// loop invariance (it emits no instruction), so the compiler cannot hoist
// base + offset into one live 64-bit pointer per row across the block loop.
// The encode reads the gradient with ordinary loads: measured faster than
// streaming loads for its c-row access pattern (the decode and the rounds
// stream with non-temporal loads, which measured faster for them).
__device__ inline v4f load_off(const float *ubase, uint32_t lane_bytes) {
    return *reinterpret_cast<const v4u4 *>(reinterpret_cast<const char *>(ubase) + lane_bytes);
}
__device__ inline v2f nt_load2_g(const float *ptr) {
    typedef __attribute__((address_space(1))) const v2u4 global_cv2f;
    return __builtin_nontemporal_load((global_cv2f *)(ptr));
}
// Stores of a row's entries: NT non-temporal, else through the caches.  (The
// choice is a compile-time one: of two stores under a condition the compiler
// makes a single cached one.)
//
// The interior encode and decode stream their rows out where these start on 16
// bytes: cached, the decode itself is up to 6 % faster, but the encode after it
// pays for the write-back (c = 16, p = 2.5M: 315 us + 389 against 332 + 334).
// Elsewhere a lane's 16 bytes straddle cache lines that its neighbours complete
// in the L2 (odd d, decode of c = 32 979 us against 1323 non-temporal, c = 64
// 1054 against 1371; odd work pointer, step-call ring of c = 64 3.60 ms against
// 4.05 with the encode non-temporal).
__device__ inline bool rows_on_16(const float *first, size_t ld) { return ld % 4 == 0 && ((uintptr_t)first & 15) == 0; }
template <bool NT>
__device__ inline void store_off(float *ubase, uint32_t lane_bytes, v4f v) {
    v4u4 *ptr = reinterpret_cast<v4u4 *>(reinterpret_cast<char *>(ubase) + lane_bytes);
    if (NT) __builtin_nontemporal_store((v4u4)v, ptr);
    else *ptr = v;
}
__device__ inline void nt_store2_off(float *ubase, uint32_t lane_bytes, v2f v) {
    __builtin_nontemporal_store((v2u4)v, reinterpret_cast<v2u4 *>(reinterpret_cast<char *>(ubase) + lane_bytes));
}

// Copies nmt M-tiles of fragments [mt][ks][lane] into LDS as [mt][ks/4][lane][ks%4].
__device__ inline void stage_fragments(float *sfrag, const float *gfrag, int nmt, int KSx) {
    const int KS4 = (KSx + 3) / 4;
    const int total = nmt * KS4 * 64 * 4;
    for (int idx = threadIdx.x; idx < total; idx += kThreads) {
        const int r = idx & 3, ln = (idx >> 2) & 63, q = (idx >> 8) % KS4, mt = (idx >> 8) / KS4;
        const int ks = q * 4 + r;
        sfrag[idx] = ks < KSx ? gfrag[((size_t)mt * KSx + ks) * 64 + ln] : 0.f;
    }
}

// One M-tile: 4 MFMA chains (one per position component t) over the K-steps.
template <int KS, bool AREG>
__device__ inline void mtile_mma(v4f (&acc)[4], const v4f (&b)[KS], const float (&av)[KS], const float *sfr,
                                 int KSx, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < (KS + 3) / 4; ++q) {
        v4f aq = {0.f, 0.f, 0.f, 0.f};
        if (!AREG && q * 4 < KSx) aq = *reinterpret_cast<const v4f *>(sfr + ((size_t)q * 64 + lane) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ks = q * 4 + r;
            if (ks < KS && ks < KSx) {
                const float a = AREG ? av[ks] : aq[r];
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[ks][0], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[ks][1], acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[ks][2], acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[ks][3], acc[3], 0, 0, 0);
            }
        }
    }
}

// Guard-free variant for the pipelined kernels: all KS K-steps run, the
// fragments in LDS are zero beyond the plan's K-steps (staged with KSpad = KS),
// so the reduction needs no runtime test and the wait counters stay exact.
template <int KS>
__device__ inline void mtile_mma_lds(v4f (&acc)[4], const v4f (&b)[KS], const float *sfr, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < (KS + 3) / 4; ++q) {
        const v4f aq = *reinterpret_cast<const v4f *>(sfr + ((size_t)q * 64 + lane) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ks = q * 4 + r;
            if (ks < KS) {
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[r], b[ks][0], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[r], b[ks][1], acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[r], b[ks][2], acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(aq[r], b[ks][3], acc[3], 0, 0, 0);
            }
        }
    }
}

// Two M-tiles at once on two-component B operands: four independent MFMA
// chains, enough to cover the MFMA result latency.
template <int KS>
__device__ inline void mtile2_mma_lds2(v4f (&acc)[2][2], const v2f (&b)[KS], const float *sfr0, const float *sfr1,
                                       int lane) {
#pragma unroll
    for (int m = 0; m < 2; ++m) acc[m][0] = acc[m][1] = v4f{0.f, 0.f, 0.f, 0.f};
    constexpr int NQ = (KS + 3) / 4;
    v4f n0 = *reinterpret_cast<const v4f *>(sfr0 + (size_t)lane * 4);
    v4f n1 = *reinterpret_cast<const v4f *>(sfr1 + (size_t)lane * 4);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const v4f a0 = n0, a1 = n1;                 // this K-quad's fragments; the next quad's load now
        if (q + 1 < NQ) {
            n0 = *reinterpret_cast<const v4f *>(sfr0 + ((size_t)(q + 1) * 64 + lane) * 4);
            n1 = *reinterpret_cast<const v4f *>(sfr1 + ((size_t)(q + 1) * 64 + lane) * 4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ks = q * 4 + r;
            if (ks < KS) {
                acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[r], b[ks][0], acc[0][0], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[r], b[ks][0], acc[1][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[r], b[ks][1], acc[0][1], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[r], b[ks][1], acc[1][1], 0, 0, 0);
            }
        }
    }
}

// Copies nmt M-tiles of fragments [mt][ks][lane] (KSx K-steps) into LDS as
// [mt][q][lane][r], ks = 4q + r, zero-padded to KSpad K-steps.
__device__ inline void stage_fragments_padded(float *sfrag, const float *gfrag, int nmt, int KSx, int KSpad) {
    const int Q = (KSpad + 3) / 4;
    const int total = nmt * Q * 256;
    for (int idx = threadIdx.x; idx < total; idx += kThreads) {
        const int r = idx & 3, ln = (idx >> 2) & 63, q = (idx >> 8) % Q, mt = (idx >> 8) / Q;
        const int ks = q * 4 + r;
        sfrag[idx] = ks < KSx ? gfrag[((size_t)mt * KSx + ks) * 64 + ln] : 0.f;
    }
}

// ---- K1: encode -----------------------------------------------------------------

struct EncParams {
    const float *grads;
    size_t ld_g;
    size_t d;
    SlotBase sb;
    const float *frag;      // N x MT x KSe x 64
    int N, c, MT, KSe;
    int mt0, mt1;           // M-tiles handled by this launch
    int wg_per_worker;
    size_t blk0, blk1;      // 64-position blocks [blk0, blk1) of every row
    size_t blk_per_wg;      // consecutive blocks each workgroup sweeps (a multiple of kWaves)
};

// Several independent instances of one plan (DDP buckets) in one launch:
// instance q owns workgroups [wg0_q, wg0_{q+1}) of the grid and brings its
// own buffers, chunk length and block range; the rest is shared.
constexpr int kMaxInst = 32;

struct EncInst {
    const float *grads;
    size_t d;
    float *work, *pool;
    size_t p, pool_stride;
    size_t blk0, blk1, blk_per_wg;
    unsigned wg0;
};

struct EncBatch {
    EncParams base;         // shared fields; the per-instance ones come from in[]
    int n;
    EncInst in[kMaxInst];
    // this workgroup's parameters, and its block index within its instance
    __device__ EncParams at(unsigned &bid) const {
        const EncInst &I = in[instance_of(in, n, blockIdx.x)];
        EncParams a = base;
        a.grads = I.grads;
        a.d = I.d;
        a.sb.work = I.work;
        a.sb.pool = I.pool;
        a.sb.p = I.p;
        a.sb.pool_stride = I.pool_stride;
        a.blk0 = I.blk0;
        a.blk1 = I.blk1;
        a.blk_per_wg = I.blk_per_wg;
        bid = blockIdx.x - I.wg0;
        return a;
    }
};

// Masked encode: tails, and c no multiple of 16.
template <int KS>
__device__ __forceinline__ void k_encode_body(const EncParams &a, unsigned bid) {
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int nmt = a.mt1 - a.mt0;
    const int KSx = a.KSe;
    const float *gfrag = a.frag + ((size_t)worker * a.MT + a.mt0) * KSx * 64;
    float av[kMaxRegTiles][KS];
#pragma unroll
    for (int mt = 0; mt < kMaxRegTiles; ++mt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            av[mt][ks] = (mt < nmt && ks < KSx) ? gfrag[((size_t)mt * KSx + ks) * 64 + lane] : 0.f;
    const float *src = a.grads + (size_t)worker * a.ld_g;
    float *dst = a.sb.work + (size_t)worker * a.sb.ld_work;
    float *x1 = a.sb.pool + (size_t)worker * a.N * a.sb.pool_stride;   // worker's first pool slot
    const size_t p = a.sb.p;
    const size_t first = a.blk0 + (size_t)wg * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    for (size_t blk = first + wave; blk < end; blk += kWaves) {
        const size_t e0 = blk * 64;
        v4f b[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int l = ks * 4 + krow;
            b[ks] = (ks < KSx && l < a.c) ? load_tile(src + (size_t)l * p, (size_t)l * p, e0, col, p, a.d)
                                          : v4f{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int mt = 0; mt < kMaxRegTiles; ++mt) {
            if (mt < nmt) {
                v4f acc[4];
                mtile_mma<KS, true>(acc, b, av[mt], nullptr, KSx, lane);
                // D fragment: lane (krow, col), register r holds output row 4 krow + r.
                const int jt = (a.mt0 + mt) * 16;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = jt + krow * 4 + r;
                    const v4f v = {acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
                    if (j < a.c) {
                        store_tile(dst + (size_t)j * p, 0, e0, col, p, p, v);
                        if (j == 0) store_tile(x1, 0, e0, col, p, p, v);
                    }
                }
            }
        }
    }
}

template <int KS>
__global__ __launch_bounds__(kThreads) void k_encode(EncParams a) { k_encode_body<KS>(a, blockIdx.x); }

template <int KS>
__global__ __launch_bounds__(kThreads) void k_encode_batch(EncBatch b) {
    unsigned bid;
    const EncParams a = b.at(bid);
    k_encode_body<KS>(a, bid);
}

// Pipelined interior encode for c <= 64 (up to 4 M-tiles): the coefficients
// stay in LDS, all M-tile accumulators stay in AGPRs, and the next block's
// loads are issued before the current block's stores, so every wave keeps
// loads in flight while its stores drain.
template <int KS, int MTMAX, int NB, bool NT>
__device__ __forceinline__ void k_encode_pipe_body(const EncParams &a, unsigned bid) {
    extern __shared__ float sfrag[];
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int MT = a.mt1 - a.mt0;                       // <= MTMAX
    const int KSx = a.KSe;
    constexpr int Q = (KS + 3) / 4;
    stage_fragments_padded(sfrag, a.frag + ((size_t)worker * a.MT + a.mt0) * KSx * 64, MT, KSx, KS);
    __syncthreads();
    const float *src = a.grads + (size_t)worker * a.ld_g;
    float *dst = a.sb.work + (size_t)worker * a.sb.ld_work;
    float *x1 = a.sb.pool + (size_t)worker * a.N * a.sb.pool_stride;
    const size_t p = a.sb.p;
    const size_t first = a.blk0 + (size_t)wg * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    // each wave takes groups of NB adjacent blocks; a group cut by `end`
    // re-reads the last block for its missing members and skips their stores
    size_t blk = first + (size_t)wave * NB;
    if (blk >= end) return;
    v4f b[NB][KS];
    auto load_group = [&](size_t g) {
        const uint32_t lane_in = opaque((uint32_t)(((size_t)krow * p + 4 * (size_t)col) * sizeof(float)));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const size_t bq = min(g + nb, end - 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) b[nb][ks] = load_off(src + bq * 64 + (size_t)(4 * min(ks, KSx - 1)) * p, lane_in);
        }
    };
    load_group(blk);
    while (true) {
        v4f acc[NB][MTMAX][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int mt = 0; mt < MTMAX; ++mt)
                if (mt < MT) mtile_mma_lds<KS>(acc[nb][mt], b[nb], sfrag + (size_t)mt * Q * 256, lane);
        const size_t next = blk + (size_t)kWaves * NB;
        if (next < end) load_group(next);
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 4 * (size_t)col) * sizeof(float)));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (blk + nb >= end) break;
            const size_t e0 = (blk + nb) * 64;
#pragma unroll
            for (int mt = 0; mt < MTMAX; ++mt) {
                if (mt < MT) {
                    const int jt = (a.mt0 + mt) * 16;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const v4f v = {acc[nb][mt][0][r], acc[nb][mt][1][r], acc[nb][mt][2][r], acc[nb][mt][3][r]};
                        store_off<NT>(dst + e0 + (size_t)(jt + r) * p, lane_out, v);   // 16 | c
                        if (jt + krow * 4 + r == 0) store_off<NT>(x1 + e0, (uint32_t)(4 * col * sizeof(float)), v);
                    }
                }
            }
        }
        if (next >= end) break;
        blk = next;
    }
}

template <int KS, int MTMAX, int NB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_encode_pipe(EncParams a) {
    if (rows_on_16(a.sb.work, a.sb.ld_work)) k_encode_pipe_body<KS, MTMAX, NB, true>(a, blockIdx.x);
    else k_encode_pipe_body<KS, MTMAX, NB, false>(a, blockIdx.x);
}

template <int KS, int MTMAX, int NB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_encode_pipe_batch(EncBatch b) {
    unsigned bid;
    const EncParams a = b.at(bid);
    if (rows_on_16(a.sb.work, a.sb.ld_work)) k_encode_pipe_body<KS, MTMAX, NB, true>(a, bid);
    else k_encode_pipe_body<KS, MTMAX, NB, false>(a, bid);
}

// Double-buffered interior encode for c = 16 MTC (up to 64): two register
// buffers of float4 B operands, so block n+1's loads are in flight during all
// of block n's MFMA work, and each M-tile's 16 output rows are stored as soon
// as the tile is done.  Two waves per SIMD in the register budget.
//
// The loop header sits after the first M-tile of a block on every path into
// it: the compiler's wait counts at the header merge the prologue with the
// back edge, and a header before the first tile made every other block wait
// for all of the previous block's stores to drain.
template <int KS, int MTC, bool ROT, bool NT>
__device__ __forceinline__ void k_encode_dbuf_body(const EncParams &a, unsigned bid) {
    extern __shared__ float sfrag[];
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int KSx = a.KSe;
    constexpr int Q = (KS + 3) / 4;
    stage_fragments_padded(sfrag, a.frag + (size_t)worker * a.MT * KSx * 64, MTC, KSx, KS);
    __syncthreads();
    const float *src = a.grads + (size_t)worker * a.ld_g;
    float *dst = a.sb.work + (size_t)worker * a.sb.ld_work;
    float *x1 = a.sb.pool + (size_t)worker * a.N * a.sb.pool_stride;
    const size_t p = a.sb.p;
    // ROT: worker w's runs of blocks start w/N of the row further on
    // (wrapping), so the workers do not sweep the same positions at the
    // same time (in-process A/B at N = 8, c = 64: encode 0.6 % faster, decode
    // equal or up to 6 % faster).  A single instance only: a batch's
    // instances have their own workgroup counts.
    const int wgr = ROT ? (wg + worker * (a.wg_per_worker / a.N)) % a.wg_per_worker : wg;
    const size_t first = a.blk0 + (size_t)wgr * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    size_t blk = first + wave;
    if (blk >= end) return;
    v4f b0[KS], b1[KS];
    auto load = [&](v4f (&b)[KS], size_t bq) {
        const uint32_t lane_in = opaque((uint32_t)(((size_t)krow * p + 4 * (size_t)col) * sizeof(float)));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[ks] = load_off(src + bq * 64 + (size_t)(4 * min(ks, KSx - 1)) * p, lane_in);
    };
    auto tile = [&](const v4f (&b)[KS], size_t bq, int mt) {
        const size_t e0 = bq * 64;
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 4 * (size_t)col) * sizeof(float)));
        v4f acc[4];
        mtile_mma_lds<KS>(acc, b, sfrag + (size_t)mt * Q * 256, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const v4f v = {acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
            store_off<NT>(dst + e0 + (size_t)(mt * 16 + r) * p, lane_out, v);
            if (mt == 0 && krow * 4 + r == 0) store_off<NT>(x1 + e0, (uint32_t)(4 * col * sizeof(float)), v);
        }
    };
    load(b0, blk);
    tile(b0, blk, 0);
    while (true) {
        size_t next = blk + kWaves;
        if (next < end) load(b1, next);
#pragma unroll
        for (int mt = 1; mt < MTC; ++mt) tile(b0, blk, mt);
        if (next >= end) break;
        blk = next;
        tile(b1, blk, 0);
        next = blk + kWaves;
        if (next < end) load(b0, next);
#pragma unroll
        for (int mt = 1; mt < MTC; ++mt) tile(b1, blk, mt);
        if (next >= end) break;
        blk = next;
        tile(b0, blk, 0);
    }
}

template <int KS, int MTC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MTC <= 2 ? 4 : 2, MTC <= 2 ? 4 : 2))) void k_encode_dbuf(EncParams a) {
    if (rows_on_16(a.sb.work, a.sb.ld_work)) k_encode_dbuf_body<KS, MTC, true, true>(a, blockIdx.x);
    else k_encode_dbuf_body<KS, MTC, true, false>(a, blockIdx.x);
}

template <int KS, int MTC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MTC <= 2 ? 4 : 2, MTC <= 2 ? 4 : 2))) void k_encode_dbuf_batch(EncBatch b) {
    unsigned bid;
    const EncParams a = b.at(bid);
    if (rows_on_16(a.sb.work, a.sb.ld_work)) k_encode_dbuf_body<KS, MTC, false, true>(a, bid);
    else k_encode_dbuf_body<KS, MTC, false, false>(a, bid);
}

// ---- K2/K3: one ring round ---------------------------------------------------
// MODE 0: x_next = recv + add            (rounds 1..N-1)
// MODE 1: x_next = (recv - sub) + add    (rounds N..c-1)
// MODE 2: x_next = recv - sub            (rounds c..L-1)
// One 16-byte element per thread, non-temporal loads and stores, and a
// one-shot grid: the fastest streaming shape measured on MI355X.

struct RoundParams {
    SlotBase sb;
    const RoundOp *ops;     // N entries of this round
    int wg_per_worker;      // of this launch, from workgroup wg0 of every row on
    size_t wg0;
};

constexpr int kRoundThreads = 256;

// One workgroup's share of a round for one worker, V 16-byte elements per
// thread, stored non-temporally if V is 1: workgroup wg covers [wg V, (wg + 1) V) x 1024 floats, V consecutive
// 1 KiB runs per wave.  p is a multiple of 4.
template <int MODE, int V = 1>
__device__ inline void round_body(const SlotBase &sb, const RoundOp &op, size_t wg) {
    const float *recv = sb.ptr(op.recv);
    const float *sub = MODE >= 1 ? sb.ptr(op.sub) : nullptr;   // aliases dst (in place)
    const float *add = MODE <= 1 ? sb.ptr(op.add) : nullptr;
    float *dst = sb.ptr(op.dst);
    const size_t p = sb.p;
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const size_t i = ((wg * V + u) * kRoundThreads + threadIdx.x) * 4;
        if (i < p) {
            v4f v = nt_load(recv + i);
            if (MODE == 0) v = v + nt_load(add + i);
            if (MODE == 2) v = v - nt_load(sub + i);
            if (MODE == 1) {
                const v4f s = nt_load(sub + i), t = nt_load(add + i);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = combine3(v[q], s[q], t[q]);
            }
            store_off<V == 1>(dst + i, 0, v);
        }
    }
}

template <int MODE, int V = 1>
__global__ __launch_bounds__(kRoundThreads) void k_round(RoundParams a) {
    const int worker = blockIdx.x / a.wg_per_worker;
    const int wg = blockIdx.x - worker * a.wg_per_worker;
    round_body<MODE, V>(a.sb, a.ops[worker], a.wg0 + wg);
}

// The same round for a batch of independent instances (buckets) in one
// launch: instance q owns workgroups [wg0, wg0 + N wgpw) and has its own
// message length and slot bases; the worker's slot ids are shared.
constexpr int kMaxBatch = 64;

struct BatchInst {
    float *work;
    float *pool;
    size_t p, pool_stride;
    unsigned wg0, wgpw;
};

struct BatchRoundParams {
    const RoundOp *ops;     // N entries of this round
    size_t ld_work;
    int Nc, c, nb;
    BatchInst b[kMaxBatch];
};

template <int MODE>
__global__ __launch_bounds__(kRoundThreads) void k_round_batch(BatchRoundParams a) {
    const BatchInst q = a.b[instance_of(a.b, a.nb, blockIdx.x)];
    const unsigned local = blockIdx.x - q.wg0;
    const int worker = (int)(local / q.wgpw);
    const SlotBase sb{q.work, a.ld_work, q.p, q.pool, q.pool_stride, a.Nc, a.c};
    round_body<MODE>(sb, a.ops[worker], local - (unsigned)worker * q.wgpw);
}

// ---- K4: decode ----------------------------------------------------------------

struct DecParams {
    SlotBase sb;
    const int *ycols;       // N x K slot ids
    float *out;
    size_t ld_o;
    size_t d;
    const float *frag;      // N x MT x KSd x 64
    int N, c, K, MT, KSd;
    int mt0, mt1;
    int wg_per_worker;
    size_t blk0, blk1;
    size_t blk_per_wg;
};

struct DecInst {
    float *work, *pool;
    size_t p, pool_stride;
    float *out;
    size_t d;
    size_t blk0, blk1, blk_per_wg;
    unsigned wg0;
};

struct DecBatch {
    DecParams base;         // shared fields; the per-instance ones come from in[]
    int n;
    DecInst in[kMaxInst];
    __device__ DecParams at(unsigned &bid) const {
        const DecInst &I = in[instance_of(in, n, blockIdx.x)];
        DecParams a = base;
        a.sb.work = I.work;
        a.sb.pool = I.pool;
        a.sb.p = I.p;
        a.sb.pool_stride = I.pool_stride;
        a.out = I.out;
        a.d = I.d;
        a.blk0 = I.blk0;
        a.blk1 = I.blk1;
        a.blk_per_wg = I.blk_per_wg;
        bid = blockIdx.x - I.wg0;
        return a;
    }
};

template <int KS, bool FAST>
__device__ __forceinline__ void k_decode_body(const DecParams &a, unsigned bid) {
    extern __shared__ float smem[];
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int nmt = a.mt1 - a.mt0;
    const int KSx = a.KSd, KS4 = (KSx + 3) / 4;
    const size_t nfrag = (size_t)nmt * KS4 * 256;
    float *sfrag = smem;
    const float **srow = reinterpret_cast<const float **>(smem + ((nfrag + 1) & ~(size_t)1));
    const float *gfrag = a.frag + ((size_t)worker * a.MT + a.mt0) * KSx * 64;
    stage_fragments(sfrag, gfrag, nmt, KSx);
    // rows K..4 KSx-1 of the last K-step repeat row K-1; their coefficients are zero
    for (int t = threadIdx.x; t < 4 * KS; t += kThreads)
        srow[t] = a.sb.ptr(a.ycols[(size_t)worker * a.K + min(t, a.K - 1)]);
    __syncthreads();
    float *out = a.out + (size_t)worker * a.ld_o;
    const size_t p = a.sb.p;
    const size_t first = a.blk0 + (size_t)wg * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    for (size_t blk = first + wave; blk < end; blk += kWaves) {
        const size_t e0 = blk * 64;
        v4f b[KS];
        if (FAST) {
            const size_t off = e0 + 4 * (size_t)col;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                b[ks] = ks < KSx ? nt_load_g(srow[ks * 4 + krow] + off) : v4f{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k = ks * 4 + krow;
                b[ks] = (ks < KSx && k < a.K) ? load_tile(srow[k], 0, e0, col, p, p) : v4f{0.f, 0.f, 0.f, 0.f};
            }
        }
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 4 * (size_t)col) * sizeof(float)));
        for (int m2 = 0; m2 < nmt; ++m2) {
            v4f acc[4];
            mtile_mma<KS, false>(acc, b, {}, sfrag + (size_t)m2 * KS4 * 256, KSx, lane);
            const int mtile = (a.mt0 + m2) * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = mtile + krow * 4 + r;
                const v4f v = {acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
                if (FAST) {
                    store_off<true>(out + e0 + (size_t)(mtile + r) * p, lane_out, v);   // m < c: 16 | c
                } else if (m < a.c) {
                    store_tile(out + (size_t)m * p, (size_t)m * p, e0, col, p, a.d, v);
                }
            }
        }
    }
}

template <int KS, bool FAST>
__global__ __launch_bounds__(kThreads) void k_decode(DecParams a) { k_decode_body<KS, FAST>(a, blockIdx.x); }

template <int KS, bool FAST>
__global__ __launch_bounds__(kThreads) void k_decode_batch(DecBatch b) {
    unsigned bid;
    const DecParams a = b.at(bid);
    k_decode_body<KS, FAST>(a, bid);
}

// Pipelined interior decode for c <= 64: same scheme, B rows through the
// per-worker table of observation slots; NB adjacent blocks per wave when
// the M-tiles are few (MTMAX <= 2), as in the encode.
template <int KS, int MTMAX, int NB, bool NT>
__device__ __forceinline__ void k_decode_pipe_body(const DecParams &a, unsigned bid) {
    extern __shared__ float smem[];
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int MT = a.mt1 - a.mt0;                       // <= MTMAX
    const int KSx = a.KSd;
    constexpr int Q = (KS + 3) / 4;
    const size_t nfrag = (size_t)MT * Q * 256;
    float *sfrag = smem;
    const float **srow = reinterpret_cast<const float **>(smem + nfrag);
    stage_fragments_padded(sfrag, a.frag + ((size_t)worker * a.MT + a.mt0) * KSx * 64, MT, KSx, KS);
    // 4 KS row pointers: rows K..4 KS-1 repeat row K-1 (zero coefficients), so
    // every load below is unconditional
    for (int t = threadIdx.x; t < 4 * KS; t += kThreads)
        srow[t] = a.sb.ptr(a.ycols[(size_t)worker * a.K + min(t, a.K - 1)]);
    __syncthreads();
    float *out = a.out + (size_t)worker * a.ld_o;
    const size_t p = a.sb.p;
    const size_t first = a.blk0 + (size_t)wg * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    size_t blk = first + (size_t)wave * NB;
    if (blk >= end) return;
    v4f b[NB][KS];
    auto load_group = [&](size_t g) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const size_t off = min(g + nb, end - 1) * 64 + 4 * col;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) b[nb][ks] = nt_load_g(srow[ks * 4 + krow] + off);
        }
    };
    load_group(blk);
    while (true) {
        v4f acc[NB][MTMAX][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int mt = 0; mt < MTMAX; ++mt)
                if (mt < MT) mtile_mma_lds<KS>(acc[nb][mt], b[nb], sfrag + (size_t)mt * Q * 256, lane);
        const size_t next = blk + (size_t)kWaves * NB;
        if (next < end) load_group(next);
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 4 * (size_t)col) * sizeof(float)));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if (blk + nb >= end) break;
            const size_t e0 = (blk + nb) * 64;
#pragma unroll
            for (int mt = 0; mt < MTMAX; ++mt) {
                if (mt < MT) {
                    const int mtile = (a.mt0 + mt) * 16;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const v4f v = {acc[nb][mt][0][r], acc[nb][mt][1][r], acc[nb][mt][2][r], acc[nb][mt][3][r]};
                        store_off<NT>(out + e0 + (size_t)(mtile + r) * p, lane_out, v);   // 16 | c
                    }
                }
            }
        }
        if (next >= end) break;
        blk = next;
    }
}

template <int KS, int MTMAX, int NB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(KS * NB <= 20 ? 3 : (KS * NB <= 32 ? 2 : 1)))) void k_decode_pipe(DecParams a) {
    if (rows_on_16(a.out, a.ld_o)) k_decode_pipe_body<KS, MTMAX, NB, true>(a, blockIdx.x);
    else k_decode_pipe_body<KS, MTMAX, NB, false>(a, blockIdx.x);
}

template <int KS, int MTMAX, int NB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(KS * NB <= 20 ? 3 : (KS * NB <= 32 ? 2 : 1)))) void k_decode_pipe_batch(DecBatch b) {
    unsigned bid;
    const DecParams a = b.at(bid);
    if (rows_on_16(a.out, a.ld_o)) k_decode_pipe_body<KS, MTMAX, NB, true>(a, bid);
    else k_decode_pipe_body<KS, MTMAX, NB, false>(a, bid);
}

// Double-buffered interior decode for c = 16 MTC (up to 64), same scheme as
// the double-buffered encode; the B rows come through the per-worker table of
// observation slots.
template <int KS, int MTC, bool ROT, bool NT>
__device__ __forceinline__ void k_decode_dbuf_body(const DecParams &a, unsigned bid) {
    extern __shared__ float smem[];
    const int worker = bid % a.N;           // workers interleaved across the grid
    const int wg = bid / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int KSx = a.KSd;
    constexpr int Q = (KS + 3) / 4;
    float *sfrag = smem;
    const float **srow = reinterpret_cast<const float **>(smem + (size_t)MTC * Q * 256);
    stage_fragments_padded(sfrag, a.frag + (size_t)worker * a.MT * KSx * 64, MTC, KSx, KS);
    // rows K..4 KS-1 repeat row K-1, whose coefficients there are zero
    for (int t = threadIdx.x; t < 4 * KS; t += kThreads)
        srow[t] = a.sb.ptr(a.ycols[(size_t)worker * a.K + min(t, a.K - 1)]);
    __syncthreads();
    float *out = a.out + (size_t)worker * a.ld_o;
    const size_t p = a.sb.p;
    // ROT: worker w's runs of blocks start w/N of the row further on
    // (wrapping), so the workers do not sweep the same positions at the
    // same time (in-process A/B at N = 8, c = 64: encode 0.6 % faster, decode
    // equal or up to 6 % faster).  A single instance only: a batch's
    // instances have their own workgroup counts.
    const int wgr = ROT ? (wg + worker * (a.wg_per_worker / a.N)) % a.wg_per_worker : wg;
    const size_t first = a.blk0 + (size_t)wgr * a.blk_per_wg, end = min(a.blk1, first + a.blk_per_wg);
    size_t blk = first + wave;
    if (blk >= end) return;
    v4f b0[KS], b1[KS];
    auto load = [&](v4f (&b)[KS], size_t bq) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[ks] = nt_load_g(srow[ks * 4 + krow] + bq * 64 + 4 * col);
    };
    auto tile = [&](const v4f (&b)[KS], size_t bq, int mt) {
        const size_t e0 = bq * 64;
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 4 * (size_t)col) * sizeof(float)));
        v4f acc[4];
        mtile_mma_lds<KS>(acc, b, sfrag + (size_t)mt * Q * 256, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const v4f v = {acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
            store_off<NT>(out + e0 + (size_t)(mt * 16 + r) * p, lane_out, v);   // 16 | c
        }
    };
    // loop header after a first M-tile on every path (see k_encode_dbuf)
    load(b0, blk);
    tile(b0, blk, 0);
    while (true) {
        size_t next = blk + kWaves;
        if (next < end) load(b1, next);
#pragma unroll
        for (int mt = 1; mt < MTC; ++mt) tile(b0, blk, mt);
        if (next >= end) break;
        blk = next;
        tile(b1, blk, 0);
        next = blk + kWaves;
        if (next < end) load(b0, next);
#pragma unroll
        for (int mt = 1; mt < MTC; ++mt) tile(b1, blk, mt);
        if (next >= end) break;
        blk = next;
        tile(b0, blk, 0);
    }
}

template <int KS, int MTC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MTC <= 2 ? 3 : 2, MTC <= 2 ? 3 : 2))) void k_decode_dbuf(DecParams a) {
    if (rows_on_16(a.out, a.ld_o)) k_decode_dbuf_body<KS, MTC, true, true>(a, blockIdx.x);
    else k_decode_dbuf_body<KS, MTC, true, false>(a, blockIdx.x);
}

template <int KS, int MTC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MTC <= 2 ? 3 : 2, MTC <= 2 ? 3 : 2))) void k_decode_dbuf_batch(DecBatch b) {
    unsigned bid;
    const DecParams a = b.at(bid);
    if (rows_on_16(a.out, a.ld_o)) k_decode_dbuf_body<KS, MTC, false, true>(a, bid);
    else k_decode_dbuf_body<KS, MTC, false, false>(a, bid);
}

// Wide decode for c = 16 MTC > 64 with more observations (K > 144) than the
// split-operand kernel (split.hip) takes: at 2(L+1)c flops per position the
// contraction is bound by the fp32 MFMA rate, so one
// wave per SIMD runs it with two register buffers of B operands: half-block
// n+1's loads are in flight while half-block n's MTC M-tiles run, and each
// tile's 16 output rows are stored as soon as it is done.  Half-blocks of 32
// positions (a float2 per lane and K-step) keep both buffers in the
// architectural registers.  The B rows come through the per-worker table of
// observation slots.
template <int KS, int MTC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_decode_wide(DecParams a) {
    static_assert(MTC % 2 == 0, "M-tiles run in pairs");
    extern __shared__ float smem[];
    const int worker = blockIdx.x % a.N;           // workers interleaved across the grid
    const int wg = blockIdx.x / a.N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int KSx = a.KSd;
    constexpr int Q = (KS + 3) / 4;
    float *sfrag = smem;
    const float **srow = reinterpret_cast<const float **>(smem + (size_t)MTC * Q * 256);
    stage_fragments_padded(sfrag, a.frag + (size_t)worker * a.MT * KSx * 64, MTC, KSx, KS);
    for (int t = threadIdx.x; t < 4 * KS; t += kThreads)
        srow[t] = a.sb.ptr(a.ycols[(size_t)worker * a.K + min(t, a.K - 1)]);
    __syncthreads();
    float *out = a.out + (size_t)worker * a.ld_o;
    const size_t p = a.sb.p;
    const size_t first = 2 * (a.blk0 + (size_t)wg * a.blk_per_wg),
                 end = 2 * min(a.blk1, a.blk0 + ((size_t)wg + 1) * a.blk_per_wg);
    size_t hb = first + wave;
    if (hb >= end) return;
    v2f b0[KS], b1[KS];
    auto load = [&](v2f (&b)[KS], size_t h) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b[ks] = nt_load2_g(srow[ks * 4 + krow] + h * 32 + 2 * col);
    };
    auto tile = [&](const v2f (&b)[KS], size_t h, int mt) {     // M-tiles mt and mt + 1
        const size_t e0 = h * 32;
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(krow * 4) * p + 2 * (size_t)col) * sizeof(float)));
        v4f acc[2][2];
        mtile2_mma_lds2<KS>(acc, b, sfrag + (size_t)mt * Q * 256, sfrag + (size_t)(mt + 1) * Q * 256, lane);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const v2f v = {acc[m][0][r], acc[m][1][r]};
                nt_store2_off(out + e0 + (size_t)((mt + m) * 16 + r) * p, lane_out, v);
            }
    };
    // the next half-block's loads go out after the first M-tile pair, when this
    // half-block's operands have all arrived.  The loop header precedes the
    // first pair, so every other half-block waits for the previous stores to
    // drain; a header after the first pair measured slower here, since the
    // third copy of the pair's code costs scalar-register spills.
    load(b0, hb);
    while (true) {
        size_t next = hb + kWaves;
        tile(b0, hb, 0);
        if (next < end) load(b1, next);
#pragma unroll
        for (int mt = 2; mt < MTC; mt += 2) tile(b0, hb, mt);
        if (next >= end) break;
        hb = next;
        next = hb + kWaves;
        tile(b1, hb, 0);
        if (next < end) load(b0, next);
#pragma unroll
        for (int mt = 2; mt < MTC; mt += 2) tile(b1, hb, mt);
        if (next >= end) break;
        hb = next;
    }
}

// ---- K5: error norms ---------------------------------------------------------

__global__ void k_fill_zero(double *x, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.0;
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Four consecutive entries of a row that starts at any float.
__device__ inline v4f row4(const float *row, size_t e, size_t d) {
    typedef float U __attribute__((ext_vector_type(4), aligned(4)));
    typedef __attribute__((address_space(1))) const U GU;
    if (e + 3 < d) return __builtin_nontemporal_load((GU *)(row + e));
    v4f v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (e + t < d) v[t] = load1_g(row + e + t);
    return v;
}

// Squared errors of W workers per grid row (blockIdx.y) against S = sum_w
// grads_w, in fp64.  Bound by memory on 2N rows: a thread takes four entries
// of every row, and the loads of eight rows are under way at a time (one
// entry per thread and row after row moved 3.8 TB/s at N = 8, d = 124M).
// Entries past d load as zero in every row and add nothing.
template <int W>
__global__ __launch_bounds__(kThreads) void k_norms(int N, size_t d, const float *__restrict__ grads,
                                                   size_t ld_g, const float *__restrict__ out, size_t ld_o,
                                                   double *norms) {
    __shared__ double red[kWaves][W + 1];
    const int w0 = blockIdx.y * W;
    double acc[W + 1];
#pragma unroll
    for (int q = 0; q <= W; ++q) acc[q] = 0.0;
    for (size_t e = 4 * ((size_t)blockIdx.x * kThreads + threadIdx.x); e < d; e += (size_t)gridDim.x * kThreads * 4) {
        double S[4] = {0.0, 0.0, 0.0, 0.0};
        for (int w = 0; w < N; w += 8) {
            v4f g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                g[q] = w + q < N ? row4(grads + (size_t)(w + q) * ld_g, e, d) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) S[t] += (double)g[q][t];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[W] += S[t] * S[t];
#pragma unroll
        for (int q0 = 0; q0 < W; q0 += 8) {
            v4f o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                o[q] = w0 + q0 + q < N ? row4(out + (size_t)(w0 + q0 + q) * ld_o, e, d) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (w0 + q0 + q < N)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const double diff = (double)o[q][t] - S[t];
                        acc[q0 + q] += diff * diff;
                    }
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q <= W; ++q) {
        const double v = wave_sum(acc[q]);
        if (lane == 0) red[wave][q] = v;
    }
    __syncthreads();
    if (threadIdx.x <= W) {
        const int q = threadIdx.x;
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += red[w][q];
        if (q < W) {
            if (w0 + q < N) atomicAdd(norms + w0 + q, v);
        } else if (blockIdx.y == 0) {
            atomicAdd(norms + N, v);
        }
    }
}

// K5's parity term: per worker w (blockIdx.y), the squared difference between
// the device outputs at sampled flat indices and reference values computed
// elsewhere, and the squared reference, in fp64.  An index outside [0, d)
// contributes NaN instead of being read.
__global__ __launch_bounds__(kThreads) void k_sampled_norms(size_t count, size_t d, const int64_t *__restrict__ idx,
                                                           const double *__restrict__ ref, const float *__restrict__ out,
                                                           size_t ld_o, double *norms) {
    __shared__ double red[kWaves][2];
    const int w = blockIdx.y;
    double dd = 0.0, rr = 0.0;
    for (size_t t = (size_t)blockIdx.x * kThreads + threadIdx.x; t < count; t += (size_t)gridDim.x * kThreads) {
        const double r = ref[(size_t)w * count + t];
        const int64_t e = idx[t];
        const double g = (e >= 0 && (uint64_t)e < d) ? (double)out[(size_t)w * ld_o + (size_t)e] : __builtin_nan("");
        const double diff = g - r;
        dd += diff * diff;
        rr += r * r;
    }
    dd = wave_sum(dd);
    rr = wave_sum(rr);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[wave][0] = dd;
        red[wave][1] = rr;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double v = 0.0;
        for (int q = 0; q < kWaves; ++q) v += red[q][threadIdx.x];
        atomicAdd(norms + 2 * w + threadIdx.x, v);
    }
}

// ---- copy ----------------------------------------------------------------------

constexpr int kCopyThreads = 64;

__global__ __launch_bounds__(kCopyThreads) void k_copy4(float *__restrict__ dst, const float *__restrict__ src, size_t n4) {
    const size_t i = (size_t)blockIdx.x * kCopyThreads + threadIdx.x;
    if (i < n4) nt_store(dst + 4 * i, nt_load(src + 4 * i));
}

__global__ void k_copy1(float *__restrict__ dst, const float *__restrict__ src, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// ---- host helpers ----------------------------------------------------------------

int hip_fail(hipError_t e, const char *what) {
    return fail(CERAR_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr, what)                         \
    do {                                            \
        hipError_t _e = (expr);                     \
        if (_e != hipSuccess) return hip_fail(_e, what); \
    } while (0)

template <class T>
int upload(T **dst, const T *src, size_t count) {
    HIP_TRY(hipMalloc((void **)dst, count * sizeof(T)), "hipMalloc (plan coefficients)");
    HIP_TRY(hipMemcpy(*dst, src, count * sizeof(T), hipMemcpyHostToDevice), "hipMemcpy (plan coefficients)");
    return CERAR_OK;
}

// Fp32 fragments and tables of the plan on the current device (uploaded once).
int device_copy(const cerar_plan *plan, const DeviceCopy **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    std::lock_guard<std::mutex> g(plan->dev_mu);
    auto it = plan->dev.find(dev);
    if (it != plan->dev.end()) {
        *out = &it->second;
        return CERAR_OK;
    }
    // The map entry comes first: once device memory is held, nothing here throws.
    DeviceCopy &dc = plan->dev[dev];
    int st = CERAR_OK;
    if (hipError_t e = hipDeviceGetAttribute(&dc.cus, hipDeviceAttributeMultiprocessorCount, dev); e != hipSuccess)
        st = hip_fail(e, "hipDeviceGetAttribute");
    if (!st)
        if (hipError_t e = prepare_passes(plan->N, plan->c, &dc.size); e != hipSuccess) st = hip_fail(e, "hipFuncGetAttributes");
    if (!st) st = upload(&dc.enc_frag, plan->enc_frag.data(), plan->enc_frag.size());
    if (!st) st = upload(&dc.dec_frag, plan->dec_frag.data(), plan->dec_frag.size());
    if (!st && !plan->enc_split.empty()) st = upload(&dc.enc_split, plan->enc_split.data(), plan->enc_split.size());
    if (!st && !plan->dec_split.empty()) st = upload(&dc.dec_split, plan->dec_split.data(), plan->dec_split.size());
    if (!st) st = upload(&dc.ycols, plan->tab.ycols.data(), plan->tab.ycols.size());
    if (!st) st = upload(&dc.rounds, plan->tab.rounds.data(), plan->tab.rounds.size());
    if (st) {
        (void)hipFree(dc.enc_frag);
        (void)hipFree(dc.dec_frag);
        (void)hipFree(dc.enc_split);
        (void)hipFree(dc.dec_split);
        (void)hipFree(dc.ycols);
        (void)hipFree(dc.rounds);
        plan->dev.erase(dev);
        return st;
    }
    *out = &dc;
    return CERAR_OK;
}

// Next expected step per workspace (cerar_encode_round ordering), with the
// plan and the gradient length the workspace's encode used.
struct Cursor {
    const cerar_plan *plan;
    int next;
    size_t d;
};
std::mutex g_cursor_mu;
std::map<const void *, Cursor> g_cursor;

bool aligned16(const void *ptr) { return ((uintptr_t)ptr & 15) == 0; }

bool overlap(const void *a, size_t abytes, const void *b, size_t bbytes) {
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + bbytes && pb < pa + abytes;
}

// Whether some row of a (N rows of n floats at stride lda) shares memory with
// some row of b.  Rows at one stride are compared modulo it, so that column
// slices of one array count as apart; other strides by their whole extents.
bool rows_overlap(const float *a, size_t lda, const float *b, size_t ldb, size_t N, size_t n) {
    if (!overlap(a, ((N - 1) * lda + n) * sizeof(float), b, ((N - 1) * ldb + n) * sizeof(float))) return false;
    if (lda != ldb) return true;
    const uintptr_t ld = lda * sizeof(float), len = n * sizeof(float);
    const uintptr_t apart = (a < b ? (uintptr_t)b - (uintptr_t)a : (uintptr_t)a - (uintptr_t)b) % ld;
    return apart < len || ld - apart < len;
}

struct Geometry {
    size_t p, pool_stride;
    bool vec;
};

int check_common(const cerar_plan *plan, size_t d, const void *work, size_t ld_work, const void *ws,
                 Geometry &g) {
    if (!plan) return fail(CERAR_E_INVAL, "plan is NULL");
    if (d == 0) return fail(CERAR_E_INVAL, "d must be > 0");
    if (!work || !ws) return fail(CERAR_E_INVAL, "work and ws must be non-NULL");
    int st = cerar_chunk_len(plan, d, &g.p, &g.pool_stride);
    if (st) return st;
    if (ld_work < (size_t)plan->c * g.p)
        return fail(CERAR_E_INVAL, "ld_work=%zu < c*p=%zu", ld_work, (size_t)plan->c * g.p);
    const size_t N = plan->N;
    if (overlap(work, ((N - 1) * ld_work + plan->c * g.p) * sizeof(float), ws,
                (size_t)plan->tab.pool_slots() * g.pool_stride * sizeof(float)))
        return fail(CERAR_E_INVAL, "work and ws overlap");
    g.vec = (g.p % 4 == 0) && (ld_work % 4 == 0) && aligned16(work) && aligned16(ws);
    return CERAR_OK;
}

SlotBase slot_base(const cerar_plan *plan, const Geometry &g, float *work, size_t ld_work, void *ws) {
    return SlotBase{work, ld_work, g.p, (float *)ws, g.pool_stride, plan->N * plan->c, plan->c};
}

// Workgroups per worker and the run of consecutive 64-position blocks each
// one sweeps: about 4 passes of its 4 waves, so that the workgroups resident
// at one time cover one compact window of positions in every row (measured
// faster on MI355X than interleaving the passes across the grid).
// One dispatch holds at most 2^31 - 1 workgroups along x and fewer than 2^32
// work-items along x (the packet's grid size is a 32-bit work-item count).
bool fits_dispatch(uint64_t wgs, unsigned threads) {
    return wgs >= 1 && wgs <= 0x7fffffffu && wgs * threads <= 0xffffffffu;
}

void wg_for(size_t nblk, int &wg_per_worker, size_t &blk_per_wg) {
    size_t w = (nblk + 4 * kWaves - 1) / (4 * kWaves);
    if (w < 1) w = 1;
    if (w > 16384) w = 16384;
    wg_per_worker = (int)w;
    blk_per_wg = (nblk + w * kWaves - 1) / (w * kWaves) * kWaves;
}

// Launch flavours: interior blocks, and the masked kernel for the rest.
enum class Path { kFast, kMasked };

// The shared fields of a single-instance launch or of a batch table.
const EncParams &shared_of(const EncParams &a) { return a; }
const EncParams &shared_of(const EncBatch &a) { return a.base; }
const DecParams &shared_of(const DecParams &a) { return a; }
const DecParams &shared_of(const DecBatch &a) { return a.base; }

template <class P>
constexpr bool kIsBatch = std::is_same_v<P, EncBatch> || std::is_same_v<P, DecBatch>;

// Each launcher starts the single-instance kernel, or its batch twin when
// given a batch table.
template <int KS, int MTMAX, int NB, class P>
void go_encode_pipe(const P &a, dim3 g, size_t l, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_encode_pipe_batch<KS, MTMAX, NB>), g, dim3(kThreads), l, s, a);
    else hipLaunchKernelGGL((k_encode_pipe<KS, MTMAX, NB>), g, dim3(kThreads), l, s, a);
}
template <int KS, int MTC, class P>
void go_encode_dbuf(const P &a, dim3 g, size_t l, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_encode_dbuf_batch<KS, MTC>), g, dim3(kThreads), l, s, a);
    else hipLaunchKernelGGL((k_encode_dbuf<KS, MTC>), g, dim3(kThreads), l, s, a);
}
template <int KS, class P>
void go_encode(const P &a, dim3 g, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_encode_batch<KS>), g, dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((k_encode<KS>), g, dim3(kThreads), 0, s, a);
}
template <int KS, int MTMAX, int NB, class P>
void go_decode_pipe(const P &a, dim3 g, size_t l, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_decode_pipe_batch<KS, MTMAX, NB>), g, dim3(kThreads), l, s, a);
    else hipLaunchKernelGGL((k_decode_pipe<KS, MTMAX, NB>), g, dim3(kThreads), l, s, a);
}
template <int KS, int MTC, class P>
void go_decode_dbuf(const P &a, dim3 g, size_t l, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_decode_dbuf_batch<KS, MTC>), g, dim3(kThreads), l, s, a);
    else hipLaunchKernelGGL((k_decode_dbuf<KS, MTC>), g, dim3(kThreads), l, s, a);
}
template <int KS, bool FAST, class P>
void go_decode(const P &a, dim3 g, size_t l, hipStream_t s) {
    if constexpr (kIsBatch<P>) hipLaunchKernelGGL((k_decode_batch<KS, FAST>), g, dim3(kThreads), l, s, a);
    else hipLaunchKernelGGL((k_decode<KS, FAST>), g, dim3(kThreads), l, s, a);
}

template <int KS, class P>
void launch_encode_ks(const P &a, Path path, hipStream_t s, dim3 grid) {
    const EncParams &sh = shared_of(a);
    if constexpr (KS >= 4) {
        if (path == Path::kFast) {
            if constexpr (KS == 16) {
                if (sh.MT == 4 && sh.mt0 == 0 && sh.mt1 == 4) {   // c = 64: double-buffered
                    go_encode_dbuf<KS, 4>(a, grid, (size_t)4 * (KS / 4) * 256 * sizeof(float), s);
                    return;
                }
            }
            if constexpr (KS == 8) {
                if (sh.MT == 2 && sh.mt0 == 0 && sh.mt1 == 2) {   // c = 32: double-buffered
                    go_encode_dbuf<KS, 2>(a, grid, (size_t)2 * (KS / 4) * 256 * sizeof(float), s);
                    return;
                }
            }
            // up to 4 M-tiles: the pipelined kernel, coefficients staged in LDS;
            // NB blocks per wave keep ~16 KB of loads in flight per wave at any c
            constexpr int MTMAX = KS <= 4 ? 1 : (KS <= 8 ? 2 : 4);
            constexpr int NB = KS <= 4 ? 4 : (KS <= 8 ? 2 : 1);
            go_encode_pipe<KS, MTMAX, NB>(a, grid, (size_t)(sh.mt1 - sh.mt0) * ((KS + 3) / 4) * 256 * sizeof(float), s);
            return;
        }
    }
    // (the interior blocks of a plan have c % 16 == 0, so KS >= 4)
    go_encode<KS>(a, grid, s);
}

template <int KS, class P>
void launch_decode_ks(const P &a, Path path, size_t lds, hipStream_t s, dim3 grid) {
    const DecParams &sh = shared_of(a);
    if constexpr (KS == 18 || KS == 20) {                // c = 64: K = 63 + N >= 65 observations
        if (path == Path::kFast && sh.MT == 4 && sh.mt0 == 0 && sh.mt1 == 4) {   // double-buffered
            go_decode_dbuf<KS, 4>(a, grid, (size_t)4 * ((KS + 3) / 4) * 256 * sizeof(float) +
                                               (size_t)4 * KS * sizeof(float *), s);
            return;
        }
    }
    if constexpr (KS == 10 || KS == 12) {                // c = 32: K = 31 + N, N <= 17
        if (path == Path::kFast && sh.MT == 2 && sh.mt0 == 0 && sh.mt1 == 2) {   // double-buffered
            go_decode_dbuf<KS, 2>(a, grid, (size_t)2 * ((KS + 3) / 4) * 256 * sizeof(float) +
                                               (size_t)4 * KS * sizeof(float *), s);
            return;
        }
    }
    if (path == Path::kFast && sh.mt1 - sh.mt0 <= kMaxRegTiles) {
        const size_t l = (size_t)(sh.mt1 - sh.mt0) * ((KS + 3) / 4) * 256 * sizeof(float) +
                         (size_t)4 * KS * sizeof(float *);
        if constexpr (KS <= 24) {
            if (sh.mt1 - sh.mt0 <= 2) {             // c <= 32: fewer accumulators, two blocks per wave if short
                go_decode_pipe<KS, 2, (KS <= 8 ? 2 : 1)>(a, grid, l, s);
                return;
            }
        }
        go_decode_pipe<KS, kMaxRegTiles, 1>(a, grid, l, s);
    }
    else if (path == Path::kFast) go_decode<KS, true>(a, grid, lds, s);
    else go_decode<KS, false>(a, grid, lds, s);
}

// M-tiles per launch so that their staged fragments fit the LDS budget.
int mtiles_per_launch(int MT, int KS, size_t extra) {
    const size_t per = (size_t)((KS + 3) / 4) * 256 * sizeof(float);
    const int n = (int)((kLdsBudget - extra) / per);
    return std::max(1, std::min(MT, n));
}

// Blocks [0, interior) need no masks: the whole 64-position block lies inside
// the chunk (e0 + 64 <= p) and inside the gradient for every chunk
// ((c-1) p + e0 + 64 <= d), and c is a multiple of 16 so every row of every
// M-tile is a real chunk; beyond them only the tail of the last block and the
// zero pad of the last chunk remain (at most a few blocks).
struct BlockSplit {
    size_t interior, total;
    bool skip_interior = false;   // the interior blocks were launched elsewhere
};

BlockSplit split_blocks(const cerar_plan *plan, size_t p, size_t d) {
    BlockSplit b;
    b.total = (p + 63) / 64;
    b.interior = 0;
    const size_t last_row = (size_t)(plan->c - 1) * p;
    // lane offsets of the fast path (up to 12 p + 64 floats) must fit 31 bits
    const bool small_rows = (12 * p + 64) * sizeof(float) < ((size_t)1 << 31);
    // the unmasked stores write all 16 rows of every M-tile: c must fill whole tiles
    if (small_rows && plan->c % 16 == 0 && d > last_row) b.interior = std::min(p, d - last_row) / 64;
    return b;
}

template <class Params, class Launch>
int launch_split(Params a, const BlockSplit &bs, size_t lds, hipStream_t s, int N, Launch launch) {
    if (bs.interior > 0 && !bs.skip_interior) {
        a.blk0 = 0;
        a.blk1 = bs.interior;
        wg_for(bs.interior, a.wg_per_worker, a.blk_per_wg);
        launch(a, Path::kFast, lds, s, dim3((unsigned)(N * a.wg_per_worker)));
    }
    if (bs.total > bs.interior) {
        a.blk0 = bs.interior;
        a.blk1 = bs.total;
        wg_for(bs.total - bs.interior, a.wg_per_worker, a.blk_per_wg);
        launch(a, Path::kMasked, lds, s, dim3((unsigned)(N * a.wg_per_worker)));
    }
    return CERAR_OK;
}

template <int KS>
int encode_ks(const EncParams &a, const BlockSplit &bs, hipStream_t s, int N) {
    return launch_split(a, bs, 0, s, N, [](const EncParams &x, Path path, size_t, hipStream_t st, dim3 g) {
        launch_encode_ks<KS>(x, path, st, g);
    });
}

template <int KS>
int decode_ks(const DecParams &a, const BlockSplit &bs, size_t lds, hipStream_t s, int N) {
    return launch_split(a, bs, lds, s, N, [](const DecParams &x, Path path, size_t l, hipStream_t st, dim3 g) {
        launch_decode_ks<KS>(x, path, l, st, g);
    });
}

// Calls f with the compiled K-step count that covers ks: the register-tile
// encode (c <= 64) and the decode.
template <class F>
void with_encode_ks(int ks, F f) {
    if (ks <= 1) f(std::integral_constant<int, 1>{});
    else if (ks <= 2) f(std::integral_constant<int, 2>{});
    else if (ks <= 4) f(std::integral_constant<int, 4>{});
    else if (ks <= 8) f(std::integral_constant<int, 8>{});
    else f(std::integral_constant<int, 16>{});
}

template <class F>
void with_decode_ks(int ks, F f) {
    if (ks <= 4) f(std::integral_constant<int, 4>{});
    else if (ks <= 8) f(std::integral_constant<int, 8>{});
    else if (ks <= 10) f(std::integral_constant<int, 10>{});
    else if (ks <= 12) f(std::integral_constant<int, 12>{});
    else if (ks <= 16) f(std::integral_constant<int, 16>{});
    else if (ks <= 18) f(std::integral_constant<int, 18>{});
    else if (ks <= 20) f(std::integral_constant<int, 20>{});
    else if (ks <= 24) f(std::integral_constant<int, 24>{});
    else if (ks <= 32) f(std::integral_constant<int, 32>{});
    else if (ks <= 36) f(std::integral_constant<int, 36>{});
    else if (ks <= 40) f(std::integral_constant<int, 40>{});
    else f(std::integral_constant<int, 48>{});
}

constexpr size_t kDecodeRowsBytes = (size_t)4 * kMaxDecodeKS * sizeof(float *) + 16;

// The fields of a launch that its instances share.
PassParams pass_params(const cerar_plan *plan, const DeviceCopy *dc, size_t ld_grads, size_t ld_work, size_t ld_out) {
    PassParams a;
    a.ld_g = ld_grads;
    a.ld_o = ld_out;
    a.ld_w = ld_work;
    a.efrag = dc->enc_frag;
    a.dfrag = dc->dec_frag;
    a.N = plan->N;
    a.c = plan->c;
    a.KSe = plan->KSe;
    a.KSd = plan->KSd;
    a.esplit = dc->enc_split;
    a.dsplit = dc->dec_split;
    a.coefs = plan->split_coefs;
    a.run = 0;
    a.n = 0;
    a.nblk = 0;
    a.ragged = ld_grads % 32 != 0 || ld_out % 32 != 0;
    return a;
}

void add_instance(PassParams &a, size_t P, const PassInst &in) {
    a.in[a.n] = in;
    a.in[a.n++].blk0 = a.nblk;
    a.nblk += (unsigned)((in.p + P - 1) / P);
    if (((uintptr_t)in.grads | (uintptr_t)in.out) % 128) a.ragged = 1;
}

// Whether the encode (decode) runs on split operands.
bool split_encode(const cerar_plan *plan) { return plan->KC > 0; }
bool split_decode(const cerar_plan *plan) { return !plan->dec_split.empty(); }

// One launch of the split encode or decode for up to kPassInst instances.
template <class Launch>
int split_launch(const cerar_plan *plan, const DeviceCopy *dc, PassParams a, const PassInst *in, int n, Launch launch,
                 hipStream_t s) {
    size_t half_blocks = 0;
    for (int q = 0; q < n; ++q) half_blocks += in[q].p / 32;
    a.run = split_run(plan->N, plan->KC, dc->cus, half_blocks);
    for (int q = 0; q < n; ++q) add_instance(a, 32 * a.run, in[q]);
    launch(a, plan->KC, s);
    HIP_TRY(hipGetLastError(), "launch split contraction");
    return CERAR_OK;
}

int enqueue_encode(const cerar_plan *plan, const DeviceCopy *dc, const Geometry &g, size_t d,
                   const float *grads, size_t ld_grads, float *work, size_t ld_work, void *ws, hipStream_t s) {
    if (split_encode(plan)) {
        const PassInst in{grads, nullptr, work, (float *)ws, d, g.p, g.pool_stride, 0};
        return split_launch(plan, dc, pass_params(plan, dc, ld_grads, ld_work, ld_work), &in, 1, launch_encode_split, s);
    }
    EncParams a;
    a.grads = grads;
    a.ld_g = ld_grads;
    a.d = d;
    a.sb = slot_base(plan, g, work, ld_work, ws);
    a.frag = dc->enc_frag;
    a.N = plan->N;
    a.c = plan->c;
    a.MT = plan->MT;
    a.KSe = plan->KSe;
    const BlockSplit bs = split_blocks(plan, g.p, d);
    const int N = plan->N, ks = plan->KSe;
    a.mt0 = 0;
    a.mt1 = plan->MT;
    // c <= 64 here: coefficients in registers
    with_encode_ks(ks, [&](auto K) { encode_ks<decltype(K)::value>(a, bs, s, N); });
    HIP_TRY(hipGetLastError(), "launch encode");
    return CERAR_OK;
}

// Workgroups per worker of a round of v 16-byte elements per thread.
size_t round_wgs(size_t p, int v = 1) {
    return std::max<size_t>(1, (p / 4 + (size_t)v * kRoundThreads - 1) / ((size_t)v * kRoundThreads));
}

int round_mode(const cerar_plan *plan, int k) {
    return (k <= plan->N - 1) ? 0 : (k + 1 <= plan->c ? 1 : 2);
}

// Messages of at most 2^21 floats take two 16-byte elements per thread:
// in-process A/B at N = 8, the rounds ran 8 % faster at p = 2^20 and 3-6 %
// faster at p = 2^21, but 3-4 % slower at p = 3.9M and 4.2M and 8 % slower
// at the Pythia-1.4B length (22.1M), where one element per thread stays.  The
// short messages are also stored through the caches, the next round reads them
// there (22.5 us against 23.5 at p = 1.0M, 41.1 against 43.8 at 2.0M; but 37.6
// against 33.5 at 2.5M, 162 against 154 at 7.8M).  So are messages at any float.
constexpr size_t kRoundTwoVectorMaxP = (size_t)1 << 21;

int enqueue_round(const cerar_plan *plan, const DeviceCopy *dc, const Geometry &g, int k, float *work,
                  size_t ld_work, void *ws, hipStream_t s) {
    const int N = plan->N, L = plan->L;
    if (k == L) return CERAR_OK;                     // the last round only relabels
    RoundParams a;
    a.sb = slot_base(plan, g, work, ld_work, ws);
    a.ops = dc->rounds + (size_t)k * N;
    const bool two = g.p <= kRoundTwoVectorMaxP || !g.vec;
    const size_t wgs = round_wgs(g.p, two ? 2 : 1);
    const bool fits = fits_dispatch((uint64_t)N * wgs, kRoundThreads);
    if (!fits && g.vec)
        return fail(CERAR_E_INVAL, "p=%zu is too long for one round launch over N=%d workers", g.p, N);
    // rows at any float have no such limit: slices of the positions
    const size_t slice = fits ? wgs : ((size_t)1 << 20);
    const int mode = round_mode(plan, k);
    for (size_t w = 0; w < wgs; w += slice) {
        a.wg0 = w;
        a.wg_per_worker = (int)std::min(slice, wgs - w);
        const dim3 grid((unsigned)(N * a.wg_per_worker));
        if (two) {
            if (mode == 0) hipLaunchKernelGGL((k_round<0, 2>), grid, dim3(kRoundThreads), 0, s, a);
            else if (mode == 1) hipLaunchKernelGGL((k_round<1, 2>), grid, dim3(kRoundThreads), 0, s, a);
            else hipLaunchKernelGGL((k_round<2, 2>), grid, dim3(kRoundThreads), 0, s, a);
        } else {
            if (mode == 0) hipLaunchKernelGGL((k_round<0>), grid, dim3(kRoundThreads), 0, s, a);
            else if (mode == 1) hipLaunchKernelGGL((k_round<1>), grid, dim3(kRoundThreads), 0, s, a);
            else hipLaunchKernelGGL((k_round<2>), grid, dim3(kRoundThreads), 0, s, a);
        }
    }
    HIP_TRY(hipGetLastError(), "launch round");
    return CERAR_OK;
}

int enqueue_decode(const cerar_plan *plan, const DeviceCopy *dc, const Geometry &g, size_t d,
                   const float *work, size_t ld_work, const void *ws, float *out, size_t ld_out, hipStream_t s) {
    if (split_decode(plan)) {
        const PassInst in{nullptr, out, const_cast<float *>(work), (float *)const_cast<void *>(ws), d, g.p, g.pool_stride, 0};
        return split_launch(plan, dc, pass_params(plan, dc, ld_out, ld_work, ld_out), &in, 1, launch_decode_split, s);
    }
    DecParams a;
    a.sb = slot_base(plan, g, const_cast<float *>(work), ld_work, const_cast<void *>(ws));
    a.ycols = dc->ycols;
    a.out = out;
    a.ld_o = ld_out;
    a.d = d;
    a.frag = dc->dec_frag;
    a.N = plan->N;
    a.c = plan->c;
    a.K = plan->L + 1;
    a.MT = plan->MT;
    a.KSd = plan->KSd;
    const BlockSplit bs = split_blocks(plan, g.p, d);
    const int N = plan->N, ks = plan->KSd;
    const size_t rows_bytes = kDecodeRowsBytes;
    BlockSplit rest = bs;
    if (plan->c == 128 && bs.interior > 0 && ks <= 48) {
        // c = 128: interior blocks on the wide kernel (all 8 M-tiles, one pass
        // over the observations), the tail below on the generic one
        DecParams w = a;
        w.mt0 = 0;
        w.mt1 = 8;
        w.blk0 = 0;
        w.blk1 = bs.interior;
        wg_for(bs.interior, w.wg_per_worker, w.blk_per_wg);
        const dim3 grid((unsigned)(N * w.wg_per_worker));
        auto lds_for = [](int K4) { return (size_t)8 * (K4 / 4) * 256 * sizeof(float) + (size_t)4 * K4 * sizeof(float *); };
        if (ks <= 40) hipLaunchKernelGGL((k_decode_wide<40, 8>), grid, dim3(kThreads), lds_for(40), s, w);
        else if (ks <= 44) hipLaunchKernelGGL((k_decode_wide<44, 8>), grid, dim3(kThreads), lds_for(44), s, w);
        else hipLaunchKernelGGL((k_decode_wide<48, 8>), grid, dim3(kThreads), lds_for(48), s, w);
        HIP_TRY(hipGetLastError(), "launch decode");
        if (bs.total == bs.interior) return CERAR_OK;
        rest.skip_interior = true;                    // only the tail blocks remain
    }
    const int step = mtiles_per_launch(plan->MT, ks, rows_bytes);
    for (int mt0 = 0; mt0 < plan->MT; mt0 += step) {
        a.mt0 = mt0;
        a.mt1 = std::min(plan->MT, mt0 + step);
        const size_t lds = (size_t)(a.mt1 - a.mt0) * ((ks + 3) / 4) * 256 * sizeof(float) + rows_bytes;
        with_decode_ks(ks, [&](auto K) { decode_ks<decltype(K)::value>(a, rest, lds, s, N); });
        HIP_TRY(hipGetLastError(), "launch decode");
    }
    return CERAR_OK;
}

// All rounds of up to kPassInst instances in one launch.
int enqueue_rounds(const cerar_plan *plan, const DeviceCopy *dc, const PassInst *in, int n, size_t ld_work,
                   hipStream_t s) {
    PassParams a = pass_params(plan, dc, ld_work, ld_work, ld_work);
    for (int q = 0; q < n; ++q) {
        PassInst r = in[q];
        r.grads = r.out = r.work;
        add_instance(a, rounds_positions(plan->N), r);
    }
    launch_rounds_pass(a, dc->cus, dc->size, s);
    HIP_TRY(hipGetLastError(), "launch rounds pass");
    return CERAR_OK;
}

// Positions of a one-pass block, or 0 where the call cannot go in one pass: the
// plan does not fit, or a block's outputs lie where another block's gradients
// are still to be read.  With `out` at `grads` itself a block reads and writes
// the same positions.  n: floats of a row that the call touches.
int one_pass_positions(const cerar_plan *plan, const float *grads, size_t ld_grads, const float *out, size_t ld_out,
                       size_t n) {
    if (!(grads == out && ld_grads == ld_out) && rows_overlap(grads, ld_grads, out, ld_out, plan->N, n)) return 0;
    return pass_positions(plan->N, plan->c);
}

// Encode, rounds and decode of one instance: in one pass where that is
// possible, else in turn.
int enqueue_ring(const cerar_plan *plan, const DeviceCopy *dc, const Geometry &g, size_t d, const float *grads,
                 size_t ld_grads, float *work, size_t ld_work, void *ws, float *out, size_t ld_out, hipStream_t s) {
    if (const int P = one_pass_positions(plan, grads, ld_grads, out, ld_out, d)) {
        PassParams a = pass_params(plan, dc, ld_grads, ld_work, ld_out);
        add_instance(a, P, PassInst{grads, out, work, (float *)ws, d, g.p, g.pool_stride, 0});
        launch_ring_pass(a, dc->cus, dc->size, s);
        HIP_TRY(hipGetLastError(), "launch ring pass");
        return CERAR_OK;
    }
    int st = enqueue_encode(plan, dc, g, d, grads, ld_grads, work, ld_work, ws, s);
    if (rounds_positions(plan->N)) {
        const PassInst in{grads, out, work, (float *)ws, d, g.p, g.pool_stride, 0};
        if (!st) st = enqueue_rounds(plan, dc, &in, 1, ld_work, s);
    } else {
        for (int k = 1; k <= plan->L && !st; ++k) st = enqueue_round(plan, dc, g, k, work, ld_work, ws, s);
    }
    if (!st) st = enqueue_decode(plan, dc, g, d, work, ld_work, ws, out, ld_out, s);
    return st;
}

int check_grads(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads, const float *work,
                size_t ld_work, const void *ws, const Geometry &g) {
    if (!grads) return fail(CERAR_E_INVAL, "grads is NULL");
    if (ld_grads < d) return fail(CERAR_E_INVAL, "ld_grads=%zu < d=%zu", ld_grads, d);
    const size_t N = plan->N;
    if ((const void *)grads == (const void *)work) {
        if (ld_grads != ld_work) return fail(CERAR_E_INVAL, "in-place encode needs ld_grads == ld_work");
    } else if (overlap(grads, ((N - 1) * ld_grads + d) * sizeof(float), work,
                       ((N - 1) * ld_work + plan->c * g.p) * sizeof(float))) {
        return fail(CERAR_E_INVAL, "grads and work overlap without being the same buffer");
    }
    if (overlap(grads, ((N - 1) * ld_grads + d) * sizeof(float), ws,
                (size_t)plan->tab.pool_slots() * g.pool_stride * sizeof(float)))
        return fail(CERAR_E_INVAL, "grads and ws overlap");
    return CERAR_OK;
}

int check_out(const cerar_plan *plan, size_t d, const float *work, size_t ld_work, const void *ws,
              const float *out, size_t ld_out, const Geometry &g) {
    if (!out) return fail(CERAR_E_INVAL, "out is NULL");
    if (ld_out < d) return fail(CERAR_E_INVAL, "ld_out=%zu < d=%zu", ld_out, d);
    const size_t N = plan->N;
    const size_t out_bytes = ((N - 1) * ld_out + d) * sizeof(float);
    if (overlap(out, out_bytes, work, ((N - 1) * ld_work + plan->c * g.p) * sizeof(float)) ||
        overlap(out, out_bytes, ws, (size_t)plan->tab.pool_slots() * g.pool_stride * sizeof(float)))
        return fail(CERAR_E_INVAL, "out overlaps work or ws");
    return CERAR_OK;
}

}  // namespace

void release_device(cerar_plan *plan) {
    std::lock_guard<std::mutex> g(plan->dev_mu);
    int cur = 0;
    bool have = hipGetDevice(&cur) == hipSuccess;
    for (auto &kv : plan->dev) {
        if (have) (void)hipSetDevice(kv.first);
        (void)hipFree(kv.second.enc_frag);
        (void)hipFree(kv.second.dec_frag);
        (void)hipFree(kv.second.enc_split);
        (void)hipFree(kv.second.dec_split);
        (void)hipFree(kv.second.ycols);
        (void)hipFree(kv.second.rounds);
    }
    if (have) (void)hipSetDevice(cur);
    plan->dev.clear();
    std::lock_guard<std::mutex> c(g_cursor_mu);
    for (auto it = g_cursor.begin(); it != g_cursor.end();)
        it = it->second.plan == plan ? g_cursor.erase(it) : std::next(it);
}

}  // namespace cerar

using namespace cerar;

namespace cerar {
namespace {

// ---- message pool of the entry point that allocates nothing -----------------
// cerar_ring_simulate_noalloc keeps its N*N message slots in this file-scope
// device array instead of a caller workspace.  Each device holds its own copy
// from the load of the library's code until the process ends.  In host code
// the array's name is not a device address: host code uses only the address
// hipGetSymbolAddress returns for the current device (scratch_address).
static __device__ __align__(256) float scratch[CERAR_NOALLOC_SCRATCH_BYTES / sizeof(float)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch[kMaxDevices];      // per device ordinal: this device's copy of `scratch`, once looked up

// Device address of the current device's `scratch`, looked up once per device
// with that device current (the first set-up or no-alloc call on it).
int scratch_address(float **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(CERAR_E_DEVICE, "device ordinal %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress (no-alloc message pool)");
        g_scratch[dev] = static_cast<float *>(ptr);
    }
    *out = g_scratch[dev];
    return CERAR_OK;
}

// The plan's device copy on the current device, without creating it (the
// upload allocates): E_STATE if cerar_plan_prepare_device has not run there.
int prepared_copy(const cerar_plan *plan, const DeviceCopy **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    std::lock_guard<std::mutex> g(plan->dev_mu);
    auto it = plan->dev.find(dev);
    if (it == plan->dev.end())
        return fail(CERAR_E_STATE, "the plan is not on device %d: call cerar_plan_prepare_device there first "
                    "(its upload allocates)", dev);
    *out = &it->second;
    return CERAR_OK;
}

}  // namespace
}  // namespace cerar

extern "C" int cerar_plan_prepare_device(const cerar_plan *plan) {
    clear_error();
    if (!plan) return fail(CERAR_E_INVAL, "plan is NULL");
    return guarded([&] {
        const DeviceCopy *dc;
        int st = device_copy(plan, &dc);
        float *pool;
        if (!st) st = scratch_address(&pool);          // set-up of the no-alloc entry point on this device
        return st;
    });
}

static int encode_round_impl(const cerar_plan *plan, int step, size_t d, const float *grads,
                             size_t ld_grads, float *work, size_t ld_work, void *ws, cerar_stream stream) {
    Geometry g;
    int st = check_common(plan, d, work, ld_work, ws, g);
    if (st) return st;
    if (step < 0 || step > plan->L) return fail(CERAR_E_INVAL, "step %d outside [0, L=%d]", step, plan->L);
    if (step == 0) {
        st = check_grads(plan, d, grads, ld_grads, work, ld_work, ws, g);
        if (st) return st;
    }
    {
        std::lock_guard<std::mutex> lk(g_cursor_mu);
        auto it = g_cursor.find(ws);
        if (step > 0 && (it == g_cursor.end() || it->second.plan != plan || it->second.next != step))
            return fail(CERAR_E_STATE, "step %d called out of order on this workspace", step);
        if (step > 0 && it->second.d != d)
            return fail(CERAR_E_STATE, "step %d with d=%zu on a workspace encoded with d=%zu", step, d, it->second.d);
    }
    const DeviceCopy *dc;
    st = device_copy(plan, &dc);
    if (st) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    st = step == 0 ? enqueue_encode(plan, dc, g, d, grads, ld_grads, work, ld_work, ws, s)
                   : enqueue_round(plan, dc, g, step, work, ld_work, ws, s);
    if (st) return st;
    std::lock_guard<std::mutex> lk(g_cursor_mu);
    g_cursor[ws] = Cursor{plan, step + 1, d};
    return CERAR_OK;
}

extern "C" int cerar_encode_round(const cerar_plan *plan, int step, size_t d, const float *grads,
                                  size_t ld_grads, float *work, size_t ld_work, void *ws, cerar_stream stream) {
    clear_error();
    return guarded([&] { return encode_round_impl(plan, step, d, grads, ld_grads, work, ld_work, ws, stream); });
}

static int decode_impl(const cerar_plan *plan, size_t d, const float *work, size_t ld_work, const void *ws,
                       float *out, size_t ld_out, cerar_stream stream) {
    Geometry g;
    int st = check_common(plan, d, work, ld_work, ws, g);
    if (st) return st;
    st = check_out(plan, d, work, ld_work, ws, out, ld_out, g);
    if (st) return st;
    {
        std::lock_guard<std::mutex> lk(g_cursor_mu);
        auto it = g_cursor.find(ws);
        if (it == g_cursor.end() || it->second.plan != plan || it->second.next != plan->L + 1)
            return fail(CERAR_E_STATE, "decode before rounds 1..L completed on this workspace");
        if (it->second.d != d)
            return fail(CERAR_E_STATE, "decode with d=%zu on a workspace encoded with d=%zu", d, it->second.d);
    }
    const DeviceCopy *dc;
    st = device_copy(plan, &dc);
    if (st) return st;
    return enqueue_decode(plan, dc, g, d, work, ld_work, ws, out, ld_out, reinterpret_cast<hipStream_t>(stream));
}

extern "C" int cerar_decode(const cerar_plan *plan, size_t d, const float *work, size_t ld_work, const void *ws,
                            float *out, size_t ld_out, cerar_stream stream) {
    clear_error();
    return guarded([&] { return decode_impl(plan, d, work, ld_work, ws, out, ld_out, stream); });
}

static int ring_simulate_impl(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                              float *work, size_t ld_work, void *ws, float *out, size_t ld_out,
                              cerar_stream stream) {
    Geometry g;
    int st = check_common(plan, d, work, ld_work, ws, g);
    if (st) return st;
    st = check_grads(plan, d, grads, ld_grads, work, ld_work, ws, g);
    if (st) return st;
    st = check_out(plan, d, work, ld_work, ws, out, ld_out, g);
    if (st) return st;
    const DeviceCopy *dc;
    st = device_copy(plan, &dc);
    if (st) return st;
    st = enqueue_ring(plan, dc, g, d, grads, ld_grads, work, ld_work, ws, out, ld_out,
                      reinterpret_cast<hipStream_t>(stream));
    if (st) return st;
    std::lock_guard<std::mutex> lk(g_cursor_mu);
    g_cursor[ws] = Cursor{plan, plan->L + 1, d};
    return CERAR_OK;
}

extern "C" int cerar_ring_simulate(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                                   float *work, size_t ld_work, void *ws, float *out, size_t ld_out,
                                   cerar_stream stream) {
    clear_error();
    return guarded([&] {
        return ring_simulate_impl(plan, d, grads, ld_grads, work, ld_work, ws, out, ld_out, stream);
    });
}

// No device or host allocation on this path: the geometry and the size check
// are host arithmetic, the plan's device copy must already exist, the pool is
// the static array, and the rest is kernel launches (no step record either).
static int ring_simulate_noalloc_impl(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                                      float *work, size_t ld_work, float *out, size_t ld_out,
                                      cerar_stream stream) {
    if (!plan) return fail(CERAR_E_INVAL, "plan is NULL");
    size_t p, stride;
    int st = cerar_chunk_len(plan, d, &p, &stride);
    if (st) return st;
    const size_t need = (size_t)plan->tab.pool_slots() * stride * sizeof(float);
    if (need > (size_t)CERAR_NOALLOC_SCRATCH_BYTES)
        return fail(CERAR_E_INVAL, "N=%d, d=%zu needs %zu bytes of message pool (N*N slots of %zu floats); "
                    "the no-alloc pool holds %zu", plan->N, d, need, stride, (size_t)CERAR_NOALLOC_SCRATCH_BYTES);
    const DeviceCopy *dc;
    st = prepared_copy(plan, &dc);
    if (st) return st;
    float *ws;
    st = scratch_address(&ws);
    if (st) return st;
    Geometry g;
    st = check_common(plan, d, work, ld_work, ws, g);
    if (st) return st;
    st = check_grads(plan, d, grads, ld_grads, work, ld_work, ws, g);
    if (st) return st;
    st = check_out(plan, d, work, ld_work, ws, out, ld_out, g);
    if (st) return st;
    st = enqueue_ring(plan, dc, g, d, grads, ld_grads, work, ld_work, ws, out, ld_out,
                      reinterpret_cast<hipStream_t>(stream));
    return st;
}

extern "C" int cerar_ring_simulate_noalloc(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                                           float *work, size_t ld_work, float *out, size_t ld_out,
                                           cerar_stream stream) {
    clear_error();
    return guarded([&] {
        return ring_simulate_noalloc_impl(plan, d, grads, ld_grads, work, ld_work, out, ld_out, stream);
    });
}

static int ring_simulate_fused_impl(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                                    float *out, size_t ld_out, cerar_stream stream) {
    if (!plan) return fail(CERAR_E_INVAL, "plan is NULL");
    if (d == 0 || !grads || !out) return fail(CERAR_E_INVAL, "d > 0 and non-NULL buffers required");
    const int N = plan->N, c = plan->c;
    if (c % 16 != 0 || c > 64) return fail(CERAR_E_INVAL, "the fused variant needs c in {16, 32, 48, 64} (c=%d)", c);
    if (N > 16) return fail(CERAR_E_INVAL, "the fused variant needs N <= 16 (N=%d)", N);
    size_t p, stride;
    int st = cerar_chunk_len(plan, d, &p, &stride);
    if (st) return st;
    if (ld_grads < d || ld_out < d) return fail(CERAR_E_INVAL, "ld_grads and ld_out must be >= d");
    if (ld_grads % 4 || ld_out % 4 || !aligned16(grads) || !aligned16(out))
        return fail(CERAR_E_INVAL, "the fused variant needs 16-byte aligned rows");
    if (overlap(grads, (((size_t)N - 1) * ld_grads + d) * sizeof(float), out,
                (((size_t)N - 1) * ld_out + d) * sizeof(float)))
        return fail(CERAR_E_INVAL, "grads and out overlap");
    const size_t lds = (size_t)N * 256 * (c + 6);        // chunks, two message buffers, four staged observations
    if (lds > 160 * 1024) return fail(CERAR_E_INVAL, "N=%d, c=%d needs %zu bytes of LDS", N, c, lds);
    const DeviceCopy *dc;
    st = device_copy(plan, &dc);
    if (st) return st;
    if (N > 8 && c > 32) return fail(CERAR_E_INVAL, "the fused variant needs c <= 32 when N > 8");
    PassParams a = pass_params(plan, dc, ld_grads, 0, ld_out);
    add_instance(a, pass_positions(N, c), PassInst{grads, out, nullptr, nullptr, d, p, 0, 0});
    launch_ring_pass(a, dc->cus, dc->size, reinterpret_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError(), "launch fused");
    return CERAR_OK;
}

extern "C" int cerar_ring_simulate_fused(const cerar_plan *plan, size_t d, const float *grads, size_t ld_grads,
                                         float *out, size_t ld_out, cerar_stream stream) {
    clear_error();
    return guarded([&] { return ring_simulate_fused_impl(plan, d, grads, ld_grads, out, ld_out, stream); });
}

extern "C" int cerar_error_norms(int N, size_t d, const float *grads, size_t ld_grads, const float *out,
                                 size_t ld_out, double *norms, cerar_stream stream) {
    clear_error();
    if (N < 1 || N > kMaxN) return fail(CERAR_E_INVAL, "N=%d outside [1, %d]", N, kMaxN);
    if (d == 0 || !grads || !out || !norms) return fail(CERAR_E_INVAL, "d > 0 and non-NULL buffers required");
    if (ld_grads < d || ld_out < d) return fail(CERAR_E_INVAL, "strides must be >= d");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_fill_zero, dim3(1), dim3(128), 0, s, norms, N + 1);
    HIP_TRY(hipGetLastError(), "launch fill");
    const size_t blocks = std::min<size_t>((d + 4 * kThreads - 1) / (4 * kThreads), 4096);
    // up to 16 workers read every gradient row once; more take a grid row per 16
    if (N <= 8)
        hipLaunchKernelGGL(k_norms<8>, dim3((unsigned)blocks), dim3(kThreads), 0, s, N, d, grads, ld_grads, out, ld_out, norms);
    else
        hipLaunchKernelGGL(k_norms<16>, dim3((unsigned)blocks, (unsigned)((N + 15) / 16)), dim3(kThreads), 0, s, N, d, grads,
                           ld_grads, out, ld_out, norms);
    HIP_TRY(hipGetLastError(), "launch norms");
    return CERAR_OK;
}

extern "C" int cerar_sampled_norms(int N, size_t count, size_t d, const int64_t *idx, const double *ref,
                                   const float *out, size_t ld_out, double *norms, cerar_stream stream) {
    clear_error();
    if (N < 1 || N > kMaxN) return fail(CERAR_E_INVAL, "N=%d outside [1, %d]", N, kMaxN);
    if (count == 0 || d == 0 || !idx || !ref || !out || !norms)
        return fail(CERAR_E_INVAL, "count > 0, d > 0 and non-NULL buffers required");
    if (ld_out < d) return fail(CERAR_E_INVAL, "ld_out=%zu < d=%zu", ld_out, d);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_fill_zero, dim3(1), dim3(128), 0, s, norms, 2 * N);
    HIP_TRY(hipGetLastError(), "launch fill");
    const size_t blocks = std::min<size_t>((count + kThreads - 1) / kThreads, 1024);
    hipLaunchKernelGGL(k_sampled_norms, dim3((unsigned)blocks, (unsigned)N), dim3(kThreads), 0, s, count, d, idx, ref,
                       out, ld_out, norms);
    HIP_TRY(hipGetLastError(), "launch sampled norms");
    return CERAR_OK;
}

extern "C" int cerar_copy_f32(float *dst, const float *src, size_t n, cerar_stream stream) {
    clear_error();
    if (!dst || !src) return fail(CERAR_E_INVAL, "NULL buffer");
    if (n == 0) return CERAR_OK;
    if (overlap(dst, n * sizeof(float), src, n * sizeof(float))) return fail(CERAR_E_INVAL, "buffers overlap");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (n % 4 == 0 && aligned16(dst) && aligned16(src)) {
        const size_t n4 = n / 4;
        const size_t blocks = (n4 + kCopyThreads - 1) / kCopyThreads;
        if (!fits_dispatch(blocks, kCopyThreads))
            return fail(CERAR_E_INVAL, "copy of %zu floats is too large for one launch", n);
        hipLaunchKernelGGL(k_copy4, dim3((unsigned)blocks), dim3(kCopyThreads), 0, s, dst, src, n4);
    } else {
        size_t blocks = std::max<size_t>(1, std::min<size_t>((n + kThreads - 1) / kThreads, 1 << 16));
        hipLaunchKernelGGL(k_copy1, dim3((unsigned)blocks), dim3(kThreads), 0, s, dst, src, n);
    }
    HIP_TRY(hipGetLastError(), "launch copy");
    return CERAR_OK;
}

namespace {

struct BucketLayout {
    size_t p, stride, work_off, ws_off;
};

int bucket_layout(const cerar_plan *plan, int nb, const size_t *len, std::vector<BucketLayout> &lay,
                  size_t &work_floats, size_t &ws_bytes) {
    if (!plan) return fail(CERAR_E_INVAL, "plan is NULL");
    if (nb < 1 || !len) return fail(CERAR_E_INVAL, "need at least one bucket");
    lay.resize(nb);
    work_floats = 0;
    ws_bytes = 0;
    for (int b = 0; b < nb; ++b) {
        if (len[b] == 0) return fail(CERAR_E_INVAL, "bucket %d is empty", b);
        BucketLayout &B = lay[b];
        B.p = ((len[b] + plan->c - 1) / plan->c + kChunkAlign - 1) / kChunkAlign * kChunkAlign;
        B.stride = (B.p + 63) / 64 * 64;
        B.work_off = work_floats;
        B.ws_off = ws_bytes;
        work_floats += (size_t)plan->c * B.p;
        ws_bytes += (size_t)plan->tab.pool_slots() * B.stride * sizeof(float);
    }
    return CERAR_OK;
}

// Kernel arguments are limited to 4 KiB.
static_assert(sizeof(EncBatch) <= 4096 && sizeof(DecBatch) <= 4096, "batch tables must fit the kernel arguments");

// One bucket's share of a batched encode or decode: its buffers and geometry.
struct BucketRef {
    const float *grads;      // encode input (bucket offset applied)
    float *out;              // decode output (bucket offset applied)
    float *work;
    void *ws;
    size_t d, p, pool_stride;
};

// Every bucket's interior blocks in as few launches as kMaxInst allows, then
// every bucket's tail blocks (masked kernels) the same way.  Set(batch, q,
// bucket, blk0, blk1) fills instance q; Launch(batch, path, grid) starts it.
template <class Batch, class Set, class Launch>
int launch_bucket_batches(const cerar_plan *plan, const std::vector<BucketRef> &bk, Batch &b, Set set,
                          Launch launch) {
    const size_t N = plan->N;
    for (int pass = 0; pass < 2; ++pass) {
        b.n = 0;
        size_t wgs = 0;
        auto flush = [&]() -> int {
            if (b.n == 0) return CERAR_OK;
            if (!fits_dispatch(wgs, kThreads)) return fail(CERAR_E_INVAL, "bucket batch too large for one launch");
            launch(b, pass == 0 ? Path::kFast : Path::kMasked, dim3((unsigned)wgs));
            HIP_TRY(hipGetLastError(), "launch bucket batch");
            b.n = 0;
            wgs = 0;
            return CERAR_OK;
        };
        for (size_t q = 0; q < bk.size(); ++q) {
            const BlockSplit bs = split_blocks(plan, bk[q].p, bk[q].d);
            const size_t lo = pass == 0 ? 0 : bs.interior, hi = pass == 0 ? bs.interior : bs.total;
            if (hi <= lo) continue;
            int wgpw;
            size_t bpw;
            wg_for(hi - lo, wgpw, bpw);
            if (b.n > 0 && !fits_dispatch(wgs + N * (size_t)wgpw, kThreads)) {
                const int st = flush();
                if (st) return st;
            }
            set(b, b.n, bk[q], lo, hi, bpw);
            b.in[b.n].wg0 = (unsigned)wgs;
            ++b.n;
            wgs += N * (size_t)wgpw;
            if (b.n == kMaxInst) {
                const int st = flush();
                if (st) return st;
            }
        }
        const int st = flush();
        if (st) return st;
    }
    return CERAR_OK;
}

int enqueue_encode_buckets(const cerar_plan *plan, const DeviceCopy *dc, const std::vector<BucketRef> &bk,
                           size_t ld_grads, size_t ld_work, hipStream_t s) {
    EncBatch b;
    EncParams &a = b.base;
    a = EncParams{};
    a.ld_g = ld_grads;
    a.sb = SlotBase{nullptr, ld_work, 0, nullptr, 0, plan->N * plan->c, plan->c};
    a.frag = dc->enc_frag;
    a.N = plan->N;
    a.c = plan->c;
    a.MT = plan->MT;
    a.KSe = plan->KSe;
    a.mt0 = 0;
    a.mt1 = plan->MT;
    auto set = [](EncBatch &x, int q, const BucketRef &r, size_t lo, size_t hi, size_t bpw) {
        EncInst &I = x.in[q];
        I.grads = r.grads;
        I.d = r.d;
        I.work = r.work;
        I.pool = (float *)r.ws;
        I.p = r.p;
        I.pool_stride = r.pool_stride;
        I.blk0 = lo;
        I.blk1 = hi;
        I.blk_per_wg = bpw;
    };
    int st = CERAR_OK;
    with_encode_ks(plan->KSe, [&](auto K) {
        st = launch_bucket_batches(plan, bk, b, set, [&](const EncBatch &x, Path path, dim3 grid) {
            launch_encode_ks<decltype(K)::value>(x, path, s, grid);
        });
    });
    return st;
}

int enqueue_decode_buckets(const cerar_plan *plan, const DeviceCopy *dc, const std::vector<BucketRef> &bk,
                           size_t ld_work, size_t ld_out, hipStream_t s) {
    DecBatch b;
    DecParams &a = b.base;
    a = DecParams{};
    a.sb = SlotBase{nullptr, ld_work, 0, nullptr, 0, plan->N * plan->c, plan->c};
    a.ycols = dc->ycols;
    a.ld_o = ld_out;
    a.frag = dc->dec_frag;
    a.N = plan->N;
    a.c = plan->c;
    a.K = plan->L + 1;
    a.MT = plan->MT;
    a.KSd = plan->KSd;
    a.mt0 = 0;
    a.mt1 = plan->MT;
    const int ks = plan->KSd;
    const size_t lds = (size_t)plan->MT * ((ks + 3) / 4) * 256 * sizeof(float) + kDecodeRowsBytes;
    auto set = [](DecBatch &x, int q, const BucketRef &r, size_t lo, size_t hi, size_t bpw) {
        DecInst &I = x.in[q];
        I.work = r.work;
        I.pool = (float *)r.ws;
        I.p = r.p;
        I.pool_stride = r.pool_stride;
        I.out = r.out;
        I.d = r.d;
        I.blk0 = lo;
        I.blk1 = hi;
        I.blk_per_wg = bpw;
    };
    int st = CERAR_OK;
    with_decode_ks(ks, [&](auto K) {
        if constexpr (decltype(K)::value <= 32)      // c <= 64: K = c + N - 1 <= 127
            st = launch_bucket_batches(plan, bk, b, set, [&](const DecBatch &x, Path path, dim3 grid) {
                launch_decode_ks<decltype(K)::value>(x, path, lds, s, grid);
            });
    });
    return st;
}

}  // namespace

static int bucketed_workspace_bytes_impl(const cerar_plan *plan, const size_t *bucket_len, int nbuckets,
                                         size_t *work_floats, size_t *ws_bytes) {
    if (!work_floats || !ws_bytes) return fail(CERAR_E_INVAL, "NULL output");
    std::vector<BucketLayout> lay;
    return bucket_layout(plan, nbuckets, bucket_len, lay, *work_floats, *ws_bytes);
}

extern "C" int cerar_bucketed_workspace_bytes(const cerar_plan *plan, const size_t *bucket_len, int nbuckets,
                                              size_t *work_floats, size_t *ws_bytes) {
    clear_error();
    return guarded([&] { return bucketed_workspace_bytes_impl(plan, bucket_len, nbuckets, work_floats, ws_bytes); });
}

static int ring_simulate_bucketed_impl(const cerar_plan *plan, int nbuckets, const size_t *bucket_off,
                                       const size_t *bucket_len, const float *grads, size_t ld_grads,
                                       float *work, size_t ld_work, void *ws, float *out, size_t ld_out,
                                       cerar_stream stream) {
    std::vector<BucketLayout> lay;
    size_t work_floats, ws_bytes;
    int st = bucket_layout(plan, nbuckets, bucket_len, lay, work_floats, ws_bytes);
    if (st) return st;
    if (!bucket_off || !grads || !work || !ws || !out) return fail(CERAR_E_INVAL, "NULL argument");
    if (ld_work < work_floats) return fail(CERAR_E_INVAL, "ld_work=%zu < %zu floats of bucket slots", ld_work, work_floats);
    size_t span = 0;
    for (int b = 0; b < nbuckets; ++b) span = std::max(span, bucket_off[b] + bucket_len[b]);
    {
        std::vector<std::pair<size_t, size_t>> iv(nbuckets);
        for (int b = 0; b < nbuckets; ++b) iv[b] = {bucket_off[b], bucket_off[b] + bucket_len[b]};
        std::sort(iv.begin(), iv.end());
        for (int b = 1; b < nbuckets; ++b)
            if (iv[b].first < iv[b - 1].second) return fail(CERAR_E_INVAL, "buckets overlap");
    }
    if (ld_grads < span || ld_out < span) return fail(CERAR_E_INVAL, "ld_grads and ld_out must cover every bucket");
    const size_t N = plan->N;
    const size_t out_bytes = ((N - 1) * ld_out + span) * sizeof(float);
    const size_t work_bytes = ((N - 1) * ld_work + work_floats) * sizeof(float);
    if (overlap(out, out_bytes, work, work_bytes) || overlap(out, out_bytes, ws, ws_bytes))
        return fail(CERAR_E_INVAL, "out overlaps work or ws");
    if (overlap(grads, ((N - 1) * ld_grads + span) * sizeof(float), work, work_bytes))
        return fail(CERAR_E_INVAL, "bucketed encode is out of place: grads and work must not overlap");
    if (overlap(work, work_bytes, ws, ws_bytes)) return fail(CERAR_E_INVAL, "work and ws overlap");
    if (overlap(grads, ((N - 1) * ld_grads + span) * sizeof(float), ws, ws_bytes))
        return fail(CERAR_E_INVAL, "grads and ws overlap");
    const DeviceCopy *dc;
    st = device_copy(plan, &dc);
    if (st) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (const int P = one_pass_positions(plan, grads, ld_grads, out, ld_out, span)) {
        // every bucket's encode, rounds and decode in one launch for up to
        // kPassInst buckets
        for (int b0 = 0; b0 < nbuckets; b0 += kPassInst) {
            PassParams a = pass_params(plan, dc, ld_grads, ld_work, ld_out);
            for (int b = b0; b < std::min(nbuckets, b0 + kPassInst); ++b)
                add_instance(a, P, PassInst{grads + bucket_off[b], out + bucket_off[b], work + lay[b].work_off,
                                            (float *)((char *)ws + lay[b].ws_off), bucket_len[b], lay[b].p,
                                            lay[b].stride, 0});
            launch_ring_pass(a, dc->cus, dc->size, s);
            HIP_TRY(hipGetLastError(), "launch ring pass");
        }
        return CERAR_OK;
    }
    // every bucket's encode, then each round once for all buckets, then every
    // bucket's decode: one stream orders them.  Up to kPassInst buckets share a
    // launch on split operands, up to kMaxInst one on fp32 operands with c <= 64
    // (interior blocks, then their tails); the fp32 decode of a wider plan gets
    // its own launches for each bucket.
    std::vector<BucketRef> bk(nbuckets);
    std::vector<PassInst> inst(nbuckets);
    for (int b = 0; b < nbuckets; ++b) {
        bk[b] = BucketRef{grads + bucket_off[b], out + bucket_off[b], work + lay[b].work_off,
                          (char *)ws + lay[b].ws_off, bucket_len[b], lay[b].p, lay[b].stride};
        inst[b] = PassInst{bk[b].grads, bk[b].out, bk[b].work, (float *)bk[b].ws, bk[b].d, bk[b].p, bk[b].pool_stride, 0};
    }
    // f(first, count) for every launch's share of the buckets
    auto each_launch = [&](auto f) {
        for (int b0 = 0; b0 < nbuckets && !st; b0 += kPassInst) st = f(&inst[b0], std::min(nbuckets - b0, kPassInst));
    };
    if (split_encode(plan))
        each_launch([&](const PassInst *in, int n) {
            return split_launch(plan, dc, pass_params(plan, dc, ld_grads, ld_work, ld_out), in, n, launch_encode_split, s);
        });
    else
        st = enqueue_encode_buckets(plan, dc, bk, ld_grads, ld_work, s);
    const int P = rounds_positions(plan->N);
    if (P)
        each_launch([&](const PassInst *in, int n) { return enqueue_rounds(plan, dc, in, n, ld_work, s); });
    for (int k = 1; k < plan->L && !st && !P; ++k) {
        for (int b0 = 0; b0 < nbuckets;) {
            BatchRoundParams a;
            a.ops = dc->rounds + (size_t)k * N;
            a.ld_work = ld_work;
            a.Nc = plan->N * plan->c;
            a.c = plan->c;
            a.nb = 0;
            size_t wgs = 0;
            // up to kMaxBatch buckets, as many as one dispatch holds
            for (; b0 < nbuckets && a.nb < kMaxBatch; ++b0) {
                const BucketLayout &B = lay[b0];
                const size_t wgpw = round_wgs(B.p);
                if (!fits_dispatch(wgs + (size_t)N * wgpw, kRoundThreads)) {
                    if (a.nb == 0) return fail(CERAR_E_INVAL, "bucket of p=%zu is too long for one round launch", B.p);
                    break;
                }
                BatchInst &I = a.b[a.nb++];
                I.work = work + B.work_off;
                I.pool = (float *)((char *)ws + B.ws_off);
                I.p = B.p;
                I.pool_stride = B.stride;
                I.wgpw = (unsigned)wgpw;
                I.wg0 = (unsigned)wgs;
                wgs += (size_t)N * wgpw;
            }
            const dim3 grid((unsigned)wgs);
            const int mode = round_mode(plan, k);
            if (mode == 0) hipLaunchKernelGGL((k_round_batch<0>), grid, dim3(kRoundThreads), 0, s, a);
            else if (mode == 1) hipLaunchKernelGGL((k_round_batch<1>), grid, dim3(kRoundThreads), 0, s, a);
            else hipLaunchKernelGGL((k_round_batch<2>), grid, dim3(kRoundThreads), 0, s, a);
            HIP_TRY(hipGetLastError(), "launch bucket round");
        }
    }
    if (st) return st;
    if (split_decode(plan))
        each_launch([&](const PassInst *in, int n) {
            return split_launch(plan, dc, pass_params(plan, dc, ld_grads, ld_work, ld_out), in, n, launch_decode_split, s);
        });
    else if (plan->MT <= kMaxRegTiles) st = enqueue_decode_buckets(plan, dc, bk, ld_work, ld_out, s);
    else
        for (int b = 0; b < nbuckets && !st; ++b)
            st = enqueue_decode(plan, dc, Geometry{lay[b].p, lay[b].stride, false}, bucket_len[b], work + lay[b].work_off, ld_work,
                                (char *)ws + lay[b].ws_off, out + bucket_off[b], ld_out, s);
    return st;
}

extern "C" int cerar_ring_simulate_bucketed(const cerar_plan *plan, int nbuckets, const size_t *bucket_off,
                                            const size_t *bucket_len, const float *grads, size_t ld_grads,
                                            float *work, size_t ld_work, void *ws, float *out, size_t ld_out,
                                            cerar_stream stream) {
    clear_error();
    return guarded([&] {
        return ring_simulate_bucketed_impl(plan, nbuckets, bucket_off, bucket_len, grads, ld_grads, work, ld_work,
                                           ws, out, ld_out, stream);
    });
}
