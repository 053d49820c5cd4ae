// Encode and decode on split operands (contracts_fp32 says for which plans not):
// the step calls, and the whole ring where it does not go in one pass.  The
// encode takes any N, the decode those whose observations fit its K-steps.
//
// Bound by memory on 2c + 1 (encode) and 2c + N - 1 (decode) rows per worker.
// A workgroup of eight waves holds its worker's split coefficients in LDS and
// sweeps a run of half-blocks (32 positions), one per wave at a time; rows
// may start at any float, c need be no multiple of 16, and the blocks that
// reach past the gradient's end take masked accesses in the same launch.
// Measured: N = 16, c = 128, d = 1e8 encode 2.74 ms, decode 2.98 ms (4.6 TB/s; a
// tail launch of 0.25 ms each is gone); N = 3, c = 100, d = 1e8 the whole ring
// 3.41 -> 1.73 ms against masked fp32 kernels.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ring_pass.hpp"
#include "split.hpp"
#include "rows.hpp"

namespace cerar {
namespace {

constexpr int kWaves = 8;

// The sum over one half-block's K-steps for M-tiles mt and mt + 1: four
// independent MFMA chains.  The LDS offsets come through opaque(), so that
// the coefficient loads, which do not change from one half-block to the next,
// are not hoisted out of the block loop (they would not fit the registers);
// the scheduling barriers keep the compiler from issuing more than one chunk
// ahead of the MFMAs.
template <int KC, bool TAIL>
__device__ inline void tile_pair(v4f (&acc)[2][2], const Split3<v8bf> (&b)[KC][2], const Split3<v4bf> (&bt)[2],
                                 const __bf16 *t0, const __bf16 *t1, int lane0) {
    const uint32_t lane = opaque((uint32_t)lane0);
#pragma unroll
    for (int m = 0; m < 2; ++m) acc[m][0] = acc[m][1] = v4f{0.f, 0.f, 0.f, 0.f};
    Split3<v8bf> a0 = tile_a32(t0, 0, lane), a1 = tile_a32(t1, 0, lane);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        Split3<v8bf> n0 = a0, n1 = a1;
        if (kc + 1 < KC) {
            n0 = tile_a32(t0, kc + 1, lane);
            n1 = tile_a32(t1, kc + 1, lane);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            acc[0][q] = mma_split32(a0, b[kc][q], acc[0][q]);
            acc[1][q] = mma_split32(a1, b[kc][q], acc[1][q]);
        }
        __builtin_amdgcn_sched_barrier(0);
        a0 = n0;
        a1 = n1;
    }
    if constexpr (TAIL) {
        const uint32_t l4 = opaque(lane);
        const Split3<v4bf> s0 = tile_a16(t0, KC, l4), s1 = tile_a16(t1, KC, l4);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            acc[0][q] = mma_split16(s0, bt[q], acc[0][q]);
            acc[1][q] = mma_split16(s1, bt[q], acc[1][q]);
        }
    }
}

// The decode of a half-block that the split does not hold (split.hpp).
CERAR_RARE void decode_rare(const float **srow, size_t p, size_t d, size_t e0, int c, int K, const float *frag, int KS,
                            float *out, int lane) {
    const size_t e = e0 + 2 * (lane & 15);
#pragma unroll 1
    for (int mt = 0; 16 * mt < c; ++mt) {
        v4f acc[1][2];
        tiles_f32(acc, 1, frag + (size_t)mt * KS * 64, KS, lane, [&](int k, int t) { return k < K ? gload1(srow[k] + e + t) : 0.f; });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 16 * mt + 4 * (lane >> 4) + r;
            const size_t flat = (size_t)j * p + e;
            if (j < c && flat < d) gstore1(out + flat, acc[0][0][r]);
            if (j < c && flat + 1 < d) gstore1(out + flat + 1, acc[0][1][r]);
        }
    }
}

// Copies a worker's split operands into LDS.
__device__ inline void stage_split(__bf16 *sa, const uint16_t *src, int count) {
    const v4u *from = reinterpret_cast<const v4u *>(src);
    v4u *to = reinterpret_cast<v4u *>(sa);
    for (int t = threadIdx.x; t < count / 8; t += 64 * kWaves) to[t] = from[t];
}

// This workgroup's instance and half-blocks.
struct Run {
    const PassInst *in;
    int worker;
    size_t first, end;
};
__device__ inline Run run_of(const PassParams &a) {
    const unsigned r = blockIdx.x / (unsigned)a.N;        // workers interleaved across the grid
    int q = 0;
    while (q + 1 < a.n && a.in[q + 1].blk0 <= r) ++q;
    const size_t first = (size_t)(r - a.in[q].blk0) * a.run;
    return {&a.in[q], (int)(blockIdx.x % (unsigned)a.N), first, min(a.in[q].p / 32, first + a.run)};
}

// EXC: c = 32 KC.  Each wave splits its half-block's rows once into
// registers, issues the next half-block's loads into the fp32 registers that
// just became free, and then runs the M-tiles.  The loop header sits after the
// split, where on every path the last memory operations issued are those
// loads, so waiting for them never drains the stores of the half-block before.
template <int KC, bool EXC, int WPE>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_encode_split(PassParams a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __bf16 *sa = reinterpret_cast<__bf16 *>(smem_raw);
    constexpr int TE = split_tile_encode(KC);
    const Run R = run_of(a);
    const PassInst &I = *R.in;
    const int N = a.N, c = EXC ? 32 * KC : a.c, w = R.worker;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g = lane >> 4;
    stage_split(sa, a.esplit + (size_t)w * 2 * KC * TE, 2 * KC * TE);
    __syncthreads();
    const float *src = I.grads + (size_t)w * a.ld_g;
    float *dst = I.work + (size_t)w * a.ld_w;
    float *x1 = I.pool + (size_t)w * N * I.pool_stride;   // worker's first pool slot
    const size_t p = I.p, d = I.d;
    size_t hb = R.first + wave;
    if (hb >= R.end) return;
    v2f x[KC][8];
    auto load = [&](size_t h) __attribute__((always_inline)) {
        const size_t ps = opaque_s(p), e0 = h * 32;
        if (p < kNarrow / 2 && (size_t)(c - 1) * ps + e0 + 32 <= d) {   // every row of it inside the gradient, short rows
            const uint32_t lane_in = opaque((uint32_t)(((size_t)(8 * g) * ps + 2 * (size_t)col) * sizeof(float)));
            const float *row = src + e0;
#pragma unroll
            for (int u = 0; u < 8 * KC; ++u) {
                    const int kc = u / 8, s = u % 8;
                    if (EXC || 32 * kc + 32 <= (int)opaque_s(c)) {
                        x[kc][s] = gload<2>(row, lane_in);
                    } else {
                        x[kc][s] = kNoRow;
                        if (32 * kc + s + 8 * (int)opaque((uint32_t)g) < c) x[kc][s] = gload<2>(row, lane_in);
                    }
                    row = step(row, s < 7 ? ps : 25 * ps);
                }
        } else {
            const int gq = (int)opaque((uint32_t)g), cq = 2 * (int)opaque((uint32_t)col);
#pragma unroll
            for (int u = 0; u < 8 * KC; ++u) {
                    const int kc = u / 8, s = u % 8;
                    const int l = 32 * kc + 8 * gq + s;
                    const size_t flat = (size_t)l * ps + e0 + cq;
                    x[kc][s] = l < c ? v2f{0.f, 0.f} : kNoRow;
                    if (l < c && flat + 1 < d) x[kc][s] = gload<2>(src + flat, 0);
                    else if (l < c && flat < d) x[kc][s][0] = gload1(src + flat);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    };
    Split3<v8bf> b[KC][2];
    const Split3<v4bf> none[2] = {};
    Contract how;                                         // kFp32: the half-block is done
    auto split = [&]() __attribute__((always_inline)) {
        SplitRange range;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
            for (int s = 0; s < 8; ++s) range.add(x[kc][s]);
#pragma unroll
            for (int q = 0; q < 2; ++q) b[kc][q] = split8([&](int s) { return x[kc][s][q]; });
        }
        how = range.contract(a.coefs, [&](auto f) __attribute__((always_inline)) {
#pragma unroll
                   for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                       for (int s = 0; s < 8; ++s) f(x[kc][s]);
               });
        if (how == kScaled)
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int q = 0; q < 2; ++q) b[kc][q] = split8([&](int s) { return kScale * x[kc][s][q]; });
        if (how != kFp32) return;
        const size_t ps = opaque_s(p), e = hb * 32 + 2 * opaque((uint32_t)col);
        const int MT = (c + 15) / 16, gq = (int)opaque((uint32_t)g);
#pragma unroll 1
        for (int mt = 0; mt < MT; ++mt) {                 // all rows are in x: in place, a tile's stores overwrite none it needs
            v4f acc[2];
            tile_f32<KC, 8 * KC>(acc, a.efrag + (size_t)(w * MT + mt) * a.KSe * 64, a.KSe, lane,
                                 [&](int kc, int s, int t) { return x[kc][s][t]; });
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 16 * mt + 4 * gq + r;
                if (j < c) gstore<2>(dst + (size_t)j * ps + e, 0, v2f{acc[0][r], acc[1][r]});
                if (j == 0) gstore<2>(x1 + e, 0, v2f{acc[0][r], acc[1][r]});
            }
        }
    };
    load(hb);
    split();
    size_t next = hb + kWaves;
    if (next < R.end) load(next);
    while (true) {
        const size_t e0 = hb * 32;
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(g * 4) * p + 2 * (size_t)col) * sizeof(float)));
        float *row = dst + e0;
        const bool narrow = p < kNarrow;
        const float back = how == kScaled ? 1.f / kScale : 1.f;
        if (how != kFp32) {
#pragma unroll
            for (int mt = 0; mt < 2 * KC; mt += 2) {
                if (EXC || 16 * mt < (int)opaque_s(c)) {
                    v4f acc[2][2];
                    tile_pair<KC, false>(acc, b, none, sa + mt * TE, sa + (mt + 1) * TE, lane);
                    const int lrow = EXC ? 0 : 16 * mt + 4 * (int)opaque((uint32_t)g);
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const v2f v = {back * acc[m][0][r], back * acc[m][1][r]};
                            if (EXC || lrow + 16 * m + r < c) {
                                if (narrow) gstore<2>(row, lane_out, v);
                                else gstore<2>(row + (size_t)(4 * (int)opaque((uint32_t)g)) * p + 2 * col, 0, v);
                                if (mt + m == 0 && r == 0 && g == 0) gstore<2>(x1 + e0, (uint32_t)(2 * col * sizeof(float)), v);
                            }
                            row = step(row, r < 3 ? p : 13 * p);
                        }
                }
            }
        } else {
            wait_all();
        }
        if (next >= R.end) break;
        hb = next;
        split();
        __builtin_amdgcn_sched_barrier(0);
        next = hb + kWaves;
        if (next < R.end) load(next);
    }
}

// The decode of K <= 32 KC + 16 observations, in the same order; the rows come
// through a table of pointers in LDS.
template <int KC, bool EXC, int WPE>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_decode_split(PassParams a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __bf16 *sa = reinterpret_cast<__bf16 *>(smem_raw);
    constexpr int TD = split_tile_decode(KC), ROWS = 32 * KC + 16;
    const float **srow = reinterpret_cast<const float **>(smem_raw + (size_t)2 * KC * TD * sizeof(__bf16));
    const Run R = run_of(a);
    const PassInst &I = *R.in;
    const int N = a.N, c = EXC ? 32 * KC : a.c, K = c + N - 1, w = R.worker;
    const int pv = w == 0 ? N - 1 : w - 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g = lane >> 4;
    const size_t p = I.p, d = I.d;
    stage_split(sa, a.dsplit + (size_t)w * 2 * KC * TD, 2 * KC * TD);
    // rows K..ROWS-1 repeat row K-1, whose coefficients there are zero
    for (int t = threadIdx.x; t < ROWS; t += 64 * kWaves) {
        const int kk = min(t, K - 1);
        srow[t] = kk < N ? I.pool + ((size_t)pv * N + kk) * I.pool_stride
                         : (kk < K - 1 ? I.work + (size_t)pv * a.ld_w + (size_t)(kk - N) * p
                                       : I.work + (size_t)w * a.ld_w + (size_t)(c - 1) * p);
    }
    __syncthreads();
    float *out = I.out + (size_t)w * a.ld_o;
    size_t hb = R.first + wave;
    if (hb >= R.end) return;
    v2f x[KC][8], xt[4];
    // the row pointers are read from LDS in every half-block (laundered
    // index): held across the loop, 36 per lane would not fit the registers
    auto load = [&](size_t h) __attribute__((always_inline)) {
        const float *const *r8 = srow + opaque((uint32_t)(8 * g));
        const float *const *r4 = srow + 32 * KC + opaque((uint32_t)(4 * g));
        const size_t e = h * 32 + 2 * col;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
            for (int s = 0; s < 8; ++s) x[kc][s] = gload_nt<2>(r8[32 * kc + s] + e);
            __builtin_amdgcn_sched_barrier(0);        // a chunk's row pointers at a time
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) xt[s] = gload_nt<2>(r4[s] + e);
    };
    Split3<v8bf> b[KC][2];
    Split3<v4bf> bt[2];
    Contract how;
    auto split = [&]() __attribute__((always_inline)) {
        SplitRange range;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
            for (int s = 0; s < 8; ++s) range.add(x[kc][s]);
#pragma unroll
            for (int q = 0; q < 2; ++q) b[kc][q] = split8([&](int s) { return x[kc][s][q]; });
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) range.add(xt[s]);
#pragma unroll
        for (int q = 0; q < 2; ++q) bt[q] = split4([&](int s) { return xt[s][q]; });
        how = range.contract(a.coefs, [&](auto f) __attribute__((always_inline)) {
#pragma unroll
                   for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                       for (int s = 0; s < 8; ++s) f(x[kc][s]);
#pragma unroll
                   for (int s = 0; s < 4; ++s) f(xt[s]);
               });
    };
    load(hb);
    split();
    size_t next = hb + kWaves;
    if (next < R.end) load(next);
    while (true) {
        const size_t e0 = hb * 32;
        const bool fast = p < kNarrow && (size_t)(c - 1) * p + e0 + 32 <= d;
        const uint32_t lane_out = opaque((uint32_t)(((size_t)(g * 4) * p + 2 * (size_t)col) * sizeof(float)));
        if (how != kUsual) {
            decode_rare(srow, p, d, e0, c, K, a.dfrag + (size_t)w * ((c + 15) / 16) * a.KSd * 64, a.KSd, out, lane);
            wait_all();
        } else {
#pragma unroll
            for (int mt = 0; mt < 2 * KC; mt += 2) {
                if (EXC || 16 * mt < (int)opaque_s(c)) {
                    v4f acc[2][2];
                    tile_pair<KC, true>(acc, b, bt, sa + mt * TD, sa + (mt + 1) * TD, lane);
                    const size_t ps = opaque_s(p);
                    float *row = out + e0 + (size_t)(16 * mt) * ps;
                    if (fast) {
                        const int lrow = EXC ? 0 : 16 * mt + 4 * (int)opaque((uint32_t)g);
#pragma unroll
                        for (int m = 0; m < 2; ++m)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (EXC || lrow + 16 * m + r < c) {
                                    const v2f v = {acc[m][0][r], acc[m][1][r]};
                                    if (a.ragged) gstore_cached<2>(row + (size_t)(16 * m + r) * ps, lane_out, v);
                                    else gstore<2>(row + (size_t)(16 * m + r) * ps, lane_out, v);
                                }
                    } else {
                        const int lrow = 16 * mt + 4 * (int)opaque((uint32_t)g);
#pragma unroll
                        for (int m = 0; m < 2; ++m)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int j = lrow + 16 * m + r;
                                const size_t flat = (size_t)j * ps + e0 + 2 * (int)opaque((uint32_t)col);
                                if (j < c && flat + 1 < d) gstore<2>(out + flat, 0, v2f{acc[m][0][r], acc[m][1][r]});
                                else if (j < c && flat < d) gstore1(out + flat, acc[m][0][r]);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                }
            }
        }
        if (next >= R.end) break;
        hb = next;
        split();
        __builtin_amdgcn_sched_barrier(0);
        next = hb + kWaves;
        if (next < R.end) load(next);
    }
}

}  // namespace

// Half-blocks per workgroup, one per wave at least: about four workgroups for
// each that a CU holds, so that each copies its coefficients once for a long
// run and the last ones to end leave little idle.
unsigned split_run(int N, int KC, int cus, size_t half_blocks) {
    const size_t target = (size_t)cus * (KC == 4 ? 4 : 8);
    const size_t run = (half_blocks * N + target - 1) / target;
    return (unsigned)(std::max<size_t>(1, (run + kWaves - 1) / kWaves) * kWaves);
}

void launch_encode_split(const PassParams &a, int KC, hipStream_t s) {
    const dim3 grid(a.nblk * (unsigned)a.N), threads(64 * kWaves);
    const size_t lds = (size_t)2 * KC * split_tile_encode(KC) * 2;
    if (KC == 2) a.c == 64 ? k_encode_split<2, true, 3><<<grid, threads, lds, s>>>(a) : k_encode_split<2, false, 3><<<grid, threads, lds, s>>>(a);
    else if (KC == 3) a.c == 96 ? k_encode_split<3, true, 2><<<grid, threads, lds, s>>>(a) : k_encode_split<3, false, 2><<<grid, threads, lds, s>>>(a);
    else a.c == 128 ? k_encode_split<4, true, 2><<<grid, threads, lds, s>>>(a) : k_encode_split<4, false, 2><<<grid, threads, lds, s>>>(a);
}

void launch_decode_split(const PassParams &a, int KC, hipStream_t s) {
    const dim3 grid(a.nblk * (unsigned)a.N), threads(64 * kWaves);
    const size_t lds = (size_t)2 * KC * split_tile_decode(KC) * 2 + (32 * KC + 16) * sizeof(float *);
    if (KC == 2) a.c == 64 ? k_decode_split<2, true, 3><<<grid, threads, lds, s>>>(a) : k_decode_split<2, false, 3><<<grid, threads, lds, s>>>(a);
    else if (KC == 3) a.c == 96 ? k_decode_split<3, true, 2><<<grid, threads, lds, s>>>(a) : k_decode_split<3, false, 2><<<grid, threads, lds, s>>>(a);
    else a.c == 128 ? k_decode_split<4, true, 2><<<grid, threads, lds, s>>>(a) : k_decode_split<4, false, 2><<<grid, threads, lds, s>>>(a);
}

}  // namespace cerar
