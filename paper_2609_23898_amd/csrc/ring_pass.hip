// The whole all-reduce in one pass over the positions (k_ring_pass).
//
// Every step of the protocol acts on each position by itself, so a workgroup
// that holds one block of positions of all N workers can encode it, run the
// L rounds of Algorithm 1 and decode it without leaving the chip.  The call
// leaves the same bytes in `work`, the workspace and `out` as the step calls
// do: every message is still written to the slot that the ownership table
// names for it, because it is an observation of the worker that receives it;
// what falls away is reading it back.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cerar_internal.hpp"
#include "device_util.hpp"
#include "ring_pass.hpp"
#include "rows.hpp"
#include "split.hpp"

namespace cerar {
namespace {

// The blocks a workgroup takes.  Workgroups go to the 8 XCDs in turn.  Where
// rows do not start on a line (a.ragged), each XCD takes a contiguous eighth
// of the blocks, and the outputs are stored through the L2: the lines that two
// blocks share are then put together there instead of going to memory in parts
// (N = 4, c = 12, odd d = 48M: 730 -> 575 us; N = 8, c = 64, odd d = 60M: 2.62
// -> 1.89 ms).  With rows on lines the plain order and streaming stores are
// faster (c = 32: 2.70 against 2.74 ms).
struct Sweep {
    unsigned first, end, step;
};
__device__ inline Sweep sweep_of(const PassParams &a) {
    if (!a.ragged || gridDim.x % 8 != 0) return {blockIdx.x, a.nblk, gridDim.x};
    const unsigned share = (a.nblk + 7) / 8, xcd = blockIdx.x % 8;
    return {xcd * share + blockIdx.x / 8, min(a.nblk, (xcd + 1) * share), gridDim.x / 8};
}

// The coefficients of a 16-row tile as MFMA A operands, one float per lane
// and K-step; K-steps past the plan's repeat its last one (the B operands
// there are zero).
template <int KS>
__device__ inline void load_frags(float (&f)[KS], const float *frag, int KSx, int lane) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = gload1(frag + (size_t)min(ks, KSx - 1) * 64 + lane);
}

// This lane's message in the next round: lane for worker w and position e
// receives from the lane of worker w - 1 at the same position.  NX = N where
// the N workers of a position sit in adjacent lanes and the exchange is a
// data-parallel move within rows of 16 lanes; NX = 0: any N, worker by
// worker across the wave, through ds_bpermute.
template <int NX>
__device__ inline float from_prev(float x, int prev_addr, bool first) {
    const int v = __float_as_int(x);
    if constexpr (NX == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xB1, 15, 15, true));   // quad_perm 1,0,3,2
    if constexpr (NX == 4) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x93, 15, 15, true));   // quad_perm 3,0,1,2
    if constexpr (NX == 8) {
        const int a = __builtin_amdgcn_mov_dpp(v, 0x121, 15, 15, true);   // row_ror:1
        const int b = __builtin_amdgcn_mov_dpp(v, 0x129, 15, 15, true);   // row_ror:9, the wrap within 8 lanes
        return __int_as_float(first ? b : a);
    }
    if constexpr (NX == 16) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x121, 15, 15, true));
    return __int_as_float(__builtin_amdgcn_ds_bpermute(prev_addr, v));
}

// The rounds of Algorithm 1 for the positions of one block.  rows: N regions
// of WS floats, worker by worker, each c rows of P encoded chunks followed by
// N - 1 free rows.  Afterwards row kk - (N - 1) holds Y column kk >= N - 1
// (the chunk last used in round kk frees its row for it) and row c + kk
// column kk < N - 1; the last column, delta_{.,c}, is already in its row.
// stale: where delta_{.,c-1} of this block goes (no observation, but the step
// calls leave it in its chunk's slot), or nullptr.
template <int NX, int P>
__device__ __forceinline__ void rounds(float *rows, int WS, int N, int c, int wave, int lane0, float *stale,
                                       size_t ld_w, size_t left) {
    const int lane = (int)opaque((uint32_t)lane0);        // the lane's place is worked out per block, not held
    const int K = c + N - 1;
    const int PW = NX ? 64 / (NX ? NX : 1) : 64 / N;      // positions per wave
    const int rw = NX ? lane % (NX ? NX : 1) : lane / PW, rp = NX ? lane / (NX ? NX : 1) : lane - rw * PW;
    const int prev_addr = NX ? 0 : 4 * (rw == 0 ? lane + (N - 1) * PW : lane - PW);
    const bool first = rw == 0;
    for (int base = wave * PW; base < P; base += N * PW) {
        const int pos = base + rp;
        if (rw >= N || pos >= P) continue;                // whole positions drop out: all N lanes of one
        float *S = rows + rw * WS + pos;
        float x = S[0];                                   // x_{rw,1} = delta_{rw,1}
        if (stale && (size_t)pos < left) gstore1(stale + (size_t)rw * ld_w + pos, S[(c - 2) * P]);
        for (int k = 1; k < N; ++k) {
            const float add = S[k * P];
            const float recv = from_prev<NX>(x, prev_addr, first);
            S[(c + k - 1) * P] = recv;                    // B_{rw,k}
            x = recv + add;
        }
        int k = N;
        constexpr int U = 4;                              // chunks read one group of rounds ahead
        if (k + U <= c) {
            float add[U], sub[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                add[u] = S[(k + u) * P];
                sub[u] = S[(k + u - N) * P];
            }
            for (; k + U <= c; k += U) {
                float nadd[U], nsub[U];
                const int kn = min(k + U, K - U);         // rows of the next group, or some that exist
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    nadd[u] = S[(kn + u) * P];
                    nsub[u] = S[(kn + u - N) * P];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float recv = from_prev<NX>(x, prev_addr, first);
                    S[(k + u - N) * P] = recv;            // D_{rw,k+u-N+1}
                    x = combine3(recv, sub[u], add[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    add[u] = nadd[u];
                    sub[u] = nsub[u];
                }
            }
        }
        for (; k < c; ++k) {
            const float sub = S[(k - N) * P], add = S[k * P];
            const float recv = from_prev<NX>(x, prev_addr, first);
            S[(k - N) * P] = recv;
            x = combine3(recv, sub, add);
        }
        for (; k < K - 1; ++k) {                          // L = K - 1
            const float sub = S[(k - N) * P];
            const float recv = from_prev<NX>(x, prev_addr, first);
            S[(k - N) * P] = recv;
            x = recv - sub;
        }
        S[(c - 2) * P] = from_prev<NX>(x, prev_addr, first);   // round L stores D_{rw,c-1}; D_{rw,c} is delta_{rw,c}
    }
}

// c <= 16 MTC chunks (EXC: c = 16 MTC), K <= 4 KSD observations, blocks of
// P = 16 V positions, one wave per worker; persistent workgroups.
//
// What bounds it: the memory system on 100-200 rows per worker, 100s of MB
// apart.  The same loads and stores alone, with neither rounds nor
// contraction, take 2.66 of 2.68 ms at N = 8, c = 32, d = 124M (4.8 TB/s; 6.03 ms
// with a launch per round) and 0.36 of 0.38 ms at c = 16, d = 2^24 (0.88 ms);
// at c = 64, d = 354M (16.3 -> 10.2 ms) the rounds and the fp32 MFMAs add up
// (they exclude each other on this chip) and bound it.
//  - The coefficients stay in registers over the whole sweep: a fragment
//    load after the stores would wait for all of them to drain (memory
//    operations of a wave complete in order).
//  - The next block's gradient rows are loaded before the rounds and arrive
//    while this block is in its rounds and its decode.
//  - V = 4 (256-byte pieces of a row) where two workgroups of that size fit a
//    CU, c <= 32; V = 2 above that (c = 64: 10.4 ms against 14.3 with V = 4,
//    whose coefficients spill).
template <int MTC, int KSD, int V, bool EXC, int MAXT, int WPE>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(WPE))) void k_ring_pass(PassParams a) {
    typedef typename Vec<V>::T VT;
    constexpr int KSE = 4 * MTC, P = 16 * V;
    extern __shared__ __align__(16) float sm[];
    const int N = a.N, c = EXC ? 16 * MTC : a.c, K = c + N - 1;
    const int KSd = a.KSd;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int WS = pass_region(N, K, P);
    const int pv = w == 0 ? N - 1 : w - 1;                // the worker whose messages w receives
    float *mine = sm + w * WS;

    VT b[KSE];
    auto load = [&](const PassInst &I, size_t e0) {
        const size_t p = opaque_s(I.p), d = I.d;
        const float *src = I.grads + (size_t)w * a.ld_g;
        // every row of the block lies inside the gradient
        const bool inside = e0 + P <= p && (size_t)(c - 1) * p + e0 + P <= d;
        if (inside && p < kNarrow) {
            const uint32_t lane_in = opaque((uint32_t)(((size_t)krow * p + V * (size_t)col) * sizeof(float)));
            const float *row = src + e0;
#pragma unroll
            for (int ks = 0; ks < KSE; ++ks) {
                if (EXC || 4 * ks + 3 < (int)opaque_s(c)) {
                    b[ks] = gload<V>(row, lane_in);
                } else {
                    b[ks] = (VT)0.f;
                    if (4 * ks + (int)opaque((uint32_t)krow) < c) b[ks] = gload<V>(row, lane_in);
                }
                row = step(row, 4 * p);
            }
        } else if (inside) {
            const int lrow = (int)opaque((uint32_t)krow);
#pragma unroll
            for (int ks = 0; ks < KSE; ++ks) {
                const int l = 4 * ks + lrow;
                b[ks] = (VT)0.f;
                if (EXC || l < c) b[ks] = gload<V>(src + (size_t)l * p + e0 + V * col, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            const int lrow = (int)opaque((uint32_t)krow), lcol = V * (int)opaque((uint32_t)col);
#pragma unroll
            for (int ks = 0; ks < KSE; ++ks) {
                const int l = 4 * ks + lrow;
                const size_t pos = e0 + lcol, flat = (size_t)l * p + pos;
#pragma unroll
                for (int t = 0; t < V; ++t) {
                    b[ks][t] = 0.f;
                    if (l < c && pos + t < p && flat + t < d) b[ks][t] = gload1(src + flat + t);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    float uf[MTC][KSE], rf[MTC][KSD];
    // delta_w = U_w^T G_w^T on this block, rows j of P positions into LDS
    auto encode = [&]() {
#pragma unroll
        for (int mt = 0; mt < MTC; ++mt) {
            v4f acc[V];
#pragma unroll
            for (int t = 0; t < V; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KSE; ++ks)
                if (EXC || 4 * ks < (int)opaque_s(c))
#pragma unroll
                    for (int t = 0; t < V; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(uf[mt][ks], b[ks][t], acc[t], 0, 0, 0);
            // register r of lane (krow, col) is chunk 16 mt + 4 krow + r at positions V col + t
            const int lrow = 16 * mt + 4 * (int)opaque((uint32_t)krow);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                VT v;
#pragma unroll
                for (int t = 0; t < V; ++t) v[t] = acc[t][r];
                if (EXC || lrow + r < c) *reinterpret_cast<VT *>(mine + (lrow + r) * P + V * col) = v;
            }
        }
    };

    int q = 0;                                            // instance of the block in b
    auto locate = [&](unsigned g) {
        while (q + 1 < a.n && a.in[q + 1].blk0 <= g) ++q;
    };
    const Sweep sw = sweep_of(a);
    unsigned g = sw.first;
    if (g >= sw.end) return;
    locate(g);
    load(a.in[q], (size_t)(g - a.in[q].blk0) * P);
#pragma unroll
    for (int mt = 0; mt < MTC; ++mt) load_frags(uf[mt], a.efrag + ((size_t)w * MTC + mt) * a.KSe * 64, a.KSe, lane);
#pragma unroll
    for (int mt = 0; mt < MTC; ++mt) load_frags(rf[mt], a.dfrag + ((size_t)w * MTC + mt) * KSd * 64, KSd, lane);
    encode();
    for (;;) {
        const PassInst &I = a.in[q];
        const size_t p = I.p, d = I.d, ps = I.pool_stride;
        const size_t e0 = (size_t)(g - I.blk0) * P;
        const bool state = I.work != nullptr, full = e0 + P <= p, narrow = p < kNarrow;
        g += sw.step;
        const bool more = g < sw.end;
        if (more) {                                       // in flight during the rounds and the decode
            locate(g);
            load(a.in[q], (size_t)(g - a.in[q].blk0) * P);
        }
        __syncthreads();
        {
            float *stale = state ? I.work + (size_t)(c - 2) * p + e0 : nullptr;
            const size_t left = p - e0;
            if (N == 8) rounds<8, P>(sm, WS, 8, c, w, lane, stale, a.ld_w, left);
            else if (N == 4) rounds<4, P>(sm, WS, 4, c, w, lane, stale, a.ld_w, left);
            else if (N == 2) rounds<2, P>(sm, WS, 2, c, w, lane, stale, a.ld_w, left);
            else if (MAXT > 512 && N == 16) rounds<16, P>(sm, WS, 16, c, w, lane, stale, a.ld_w, left);
            else rounds<0, P>(sm, WS, N, c, w, lane, stale, a.ld_w, left);
        }
        __syncthreads();
        // decode: ghat_w = Y_w R_w; the observations to their slots: column kk
        // of Y_w is message kk + 1 of worker pv, in pv's pool for kk < N and
        // in pv's freed chunks after that; the last column is w's own last chunk
        v4f dacc[MTC][V];
#pragma unroll
        for (int mt = 0; mt < MTC; ++mt)
#pragma unroll
            for (int t = 0; t < V; ++t) dacc[mt][t] = v4f{0.f, 0.f, 0.f, 0.f};
        float *own = I.work + (size_t)w * a.ld_w + (size_t)(c - 1) * p + e0;
        float *rcv = I.work + (size_t)pv * a.ld_w + e0;
        float *pool = I.pool + (size_t)pv * N * ps + e0;
        const uint32_t lane_row = opaque((uint32_t)(((size_t)krow * p + V * (size_t)col) * sizeof(float)));
        float *row4 = step(rcv, (size_t)0) - (size_t)N * p;   // column 4 ks, for 4 ks >= N
        const float *yin = mine + (krow - (N - 1)) * P + V * col;
#pragma unroll
        for (int ks = 0; ks < KSD; ++ks) {
            const int Nq = (int)opaque_s(N), Kq = (int)opaque_s(K);   // compared here, not held as masks
            VT y = (VT)0.f;                               // rows past L meet zero coefficients
            if (narrow && 4 * ks >= Nq && 4 * ks + 3 < Kq - 1) {      // most K-steps lie in the columns N..K-2 as a whole
                y = *reinterpret_cast<const VT *>(yin + 4 * ks * P);
                if (state && full) gstore<V>(row4, lane_row, y);
            } else if (4 * ks < Kq) {
                const int kk = 4 * ks + (int)opaque((uint32_t)krow);
                if (kk < K) y = *reinterpret_cast<const VT *>(mine + (kk - (N - 1) + (kk < N - 1 ? K : 0)) * P + V * col);
                if (state && full && kk < K) {
                    float *row = kk < N ? pool + (size_t)kk * ps : (kk < K - 1 ? rcv + (size_t)(kk - N) * p : own);
                    gstore<V>(row, (uint32_t)(V * col * sizeof(float)), y);
                }
            }
            row4 = step(row4, 4 * p);
            if (4 * ks < Kq)
#pragma unroll
                for (int mt = 0; mt < MTC; ++mt)
#pragma unroll
                    for (int t = 0; t < V; ++t)
                        dacc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(rf[mt][ks], y[t], dacc[mt][t], 0, 0, 0);
        }
        if (state && !full) {                             // the last block of a row where p is no multiple of P
            for (int kk = krow; kk < K; kk += 4) {
                const float *yr = mine + (kk - (N - 1) + (kk < N - 1 ? K : 0)) * P + V * col;
                float *row = kk < N ? pool + (size_t)kk * ps : (kk < K - 1 ? rcv + (size_t)(kk - N) * p : own);
                for (int t = 0; t < V; ++t)
                    if (e0 + V * col + t < p) gstore1(row + V * col + t, yr[t]);
            }
        }
        float *out = I.out + (size_t)w * a.ld_o;
        const bool inside = full && (size_t)(c - 1) * p + e0 + P <= d;
        if (inside && narrow) {
            const uint32_t lane_out = opaque((uint32_t)(((size_t)(4 * krow) * p + V * (size_t)col) * sizeof(float)));
            float *row = out + e0;
            const bool ragged = a.ragged;
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt) {
                const int lrow = EXC ? 0 : 4 * (int)opaque((uint32_t)krow);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    VT v;
#pragma unroll
                    for (int t = 0; t < V; ++t) v[t] = dacc[mt][t][r];
                    if (EXC || 16 * mt + lrow + r < c) {
                        if (ragged) gstore_cached<V>(row, lane_out, v);
                        else gstore<V>(row, lane_out, v);
                    }
                    row = step(row, r < 3 ? p : 13 * p);
                }
            }
        } else if (inside) {
            const size_t pq = opaque_s(p);
            const int lrow = 4 * (int)opaque((uint32_t)krow);
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + lrow + r;
                    VT v;
#pragma unroll
                    for (int t = 0; t < V; ++t) v[t] = dacc[mt][t][r];
                    if (EXC || m < c) gstore<V>(out + (size_t)m * pq + e0 + V * col, 0, v);
                    __builtin_amdgcn_sched_barrier(0);
                }
        } else {
            const size_t pq = opaque_s(p);
            const int lrow = 4 * (int)opaque((uint32_t)krow), lcol = V * (int)opaque((uint32_t)col);
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + lrow + r;
                    const size_t pos = e0 + lcol, flat = (size_t)m * pq + pos;
#pragma unroll
                    for (int t = 0; t < V; ++t)
                        if (m < c && pos + t < pq && flat + t < d) gstore1(out + flat + t, dacc[mt][t][r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        if (!more) break;
        encode();                                         // reads and writes this wave's own rows only
    }
}

// The same for 8 < N <= 16 and 32 < c <= 64 (EXC: c = 64; K = c + N - 1 <= 80):
// sixteen waves leave each 128 registers, too few for the coefficients, so
// they come from the L2 for every block, split into bf16 terms (51 KB per
// worker at c = 64), and the contractions run on split operands, at 3/8 of the
// fp32 MFMA time.  Blocks of 32 positions.  N = 16, c = 60, odd d = 20M: 2.06
// -> 1.42 ms against encode, rounds and decode in turn; N = 12, c = 48, d = 40M:
// 2.88 -> 2.27 ms.  Not for N <= 8, where k_ring_pass keeps the coefficients
// (N = 8, c = 64, d = 354M: 10.4 ms there, 11.8-13.4 ms here).
__device__ inline Split3<v8bf> global_a32(const __bf16 *tile, int kc, uint32_t lane) {
    typedef __attribute__((address_space(1))) const v8bf G;
    const __bf16 *b = tile + (size_t)kc * 3 * 64 * 8 + lane * 8;
    return {*(G *)b, *(G *)(b + 64 * 8), *(G *)(b + 2 * 64 * 8)};
}
__device__ inline Split3<v4bf> global_a16(const __bf16 *tile, int KC, uint32_t lane) {
    typedef __attribute__((address_space(1))) const v4bf G;
    const __bf16 *b = tile + (size_t)KC * 3 * 64 * 8 + lane * 4;
    return {*(G *)b, *(G *)(b + 64 * 4), *(G *)(b + 2 * 64 * 4)};
}

// The encode of a block that the split does not hold (split.hpp): its gradient
// rows are read again, and the chunks go to LDS.
CERAR_RARE void encode_rare(const float *src, size_t p, size_t d, size_t e0, int c, const float *frag, int KS, float *mine,
                            int lane) {
    const size_t e = e0 + 2 * (lane & 15);
#pragma unroll 1
    for (int mt = 0; 16 * mt < c; ++mt) {
        v4f acc[2];
        tile_f32<2, 1>(acc, frag + (size_t)mt * KS * 64, KS, lane, [&](int kc, int s, int t) {
            const int l = 32 * kc + 8 * (lane >> 4) + s;
            return l < c && (size_t)l * p + e + t < d ? gload1(src + (size_t)l * p + e + t) : 0.f;
        });
        const int row0 = 16 * mt + 4 * (lane >> 4);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (row0 + r < c) *reinterpret_cast<v2f *>(mine + (row0 + r) * 32 + 2 * (lane & 15)) = v2f{acc[0][r], acc[1][r]};
    }
}

template <bool EXC>
__global__ __launch_bounds__(1024) void k_ring_pass_split(PassParams a) {
    constexpr int KC = 2, MTC = 4, P = 32, TE = split_tile_encode(KC), TD = split_tile_decode(KC);
    extern __shared__ __align__(16) float sm[];
    const int N = a.N, c = EXC ? 64 : a.c, K = c + N - 1, MT = (c + 15) / 16;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g4 = lane >> 4;
    const int WS = pass_region(N, K, P);
    const int pv = w == 0 ? N - 1 : w - 1;                // the worker whose messages w receives
    float *mine = sm + w * WS;
    const __bf16 *et = reinterpret_cast<const __bf16 *>(a.esplit) + (size_t)w * MTC * TE;
    const __bf16 *dt = reinterpret_cast<const __bf16 *>(a.dsplit) + (size_t)w * MTC * TD;

    v2f x[KC][8];                                         // rows 32 kc + 8 g4 + s at positions 2 col, 2 col + 1
    auto load = [&](const PassInst &I, size_t e0) __attribute__((always_inline)) {
        const size_t p = opaque_s(I.p), d = I.d;
        const float *src = I.grads + (size_t)w * a.ld_g;
        if (p < kNarrow / 2 && (size_t)(c - 1) * p + e0 + P <= d) {   // every row of it inside the gradient, short rows
            const uint32_t lane_in = opaque((uint32_t)(((size_t)(8 * g4) * p + 2 * (size_t)col) * sizeof(float)));
            const float *row = src + e0;
#pragma unroll
            for (int u = 0; u < 8 * KC; ++u) {
                const int kc = u / 8, s = u % 8;
                if (EXC || 32 * kc + 32 <= (int)opaque_s(c)) {
                    x[kc][s] = gload<2>(row, lane_in);
                } else {
                    x[kc][s] = kNoRow;
                    if (32 * kc + s + 8 * (int)opaque((uint32_t)g4) < c) x[kc][s] = gload<2>(row, lane_in);
                }
                row = step(row, s < 7 ? p : 25 * p);
            }
        } else {
            const int gq = (int)opaque((uint32_t)g4), cq = 2 * (int)opaque((uint32_t)col);
#pragma unroll
            for (int u = 0; u < 8 * KC; ++u) {
                const int kc = u / 8, s = u % 8;
                const int l = 32 * kc + 8 * gq + s;
                const size_t flat = (size_t)l * p + e0 + cq;
                x[kc][s] = l < c ? v2f{0.f, 0.f} : kNoRow;
                if (l < c && flat + 1 < d) x[kc][s] = gload<2>(src + flat, 0);
                else if (l < c && flat < d) x[kc][s][0] = gload1(src + flat);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // delta_w on this block, rows j of P positions into LDS
    auto encode = [&](const PassInst &I, size_t e0) __attribute__((always_inline)) {
        SplitRange range;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int s = 0; s < 8; ++s) range.add(x[kc][s]);
        const Contract how = range.contract(a.coefs, [&](auto f) __attribute__((always_inline)) {
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int s = 0; s < 8; ++s) f(x[kc][s]);
        });
        if (how == kFp32) {
            encode_rare(I.grads + (size_t)w * a.ld_g, I.p, I.d, e0, c, a.efrag + (size_t)w * MT * a.KSe * 64, a.KSe, mine, lane);
            return;
        }
        if (how == kScaled)
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int s = 0; s < 8; ++s) x[kc][s] *= kScale;
        const float back = how == kScaled ? 1.f / kScale : 1.f;
        Split3<v8bf> b[KC][2];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int q = 0; q < 2; ++q) b[kc][q] = split8([&](int s) { return x[kc][s][q]; });
        Split3<v8bf> next = global_a32(et, 0, lane);
#pragma unroll 1
        for (int mt = 0; mt < MTC; ++mt) {
            v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const Split3<v8bf> A = next;
                const bool last = kc + 1 == KC;           // then the next tile's first chunk (or this one's again)
                next = global_a32(et + (size_t)(last ? min(mt + 1, MTC - 1) : mt) * TE, last ? 0 : kc + 1, lane);
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[q] = mma_split32(A, b[kc][q], acc[q]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int lrow = 16 * mt + 4 * (int)opaque((uint32_t)g4);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (EXC || lrow + r < c)
                    *reinterpret_cast<v2f *>(mine + (lrow + r) * P + 2 * col) = v2f{back * acc[0][r], back * acc[1][r]};
        }
    };

    int q = 0;                                            // instance of the block in x
    auto locate = [&](unsigned g) {
        while (q + 1 < a.n && a.in[q + 1].blk0 <= g) ++q;
    };
    const Sweep sw = sweep_of(a);
    unsigned g = sw.first;
    if (g >= sw.end) return;
    locate(g);
    load(a.in[q], (size_t)(g - a.in[q].blk0) * P);
    encode(a.in[q], (size_t)(g - a.in[q].blk0) * P);
    for (;;) {
        const PassInst &I = a.in[q];
        const size_t p = I.p, d = I.d, ps = I.pool_stride;
        const size_t e0 = (size_t)(g - I.blk0) * P;       // p is a multiple of P: every block is a whole one
        const bool state = I.work != nullptr;
        g += sw.step;
        const bool more = g < sw.end;
        if (more) {                                       // in flight during the rounds and the decode
            locate(g);
            load(a.in[q], (size_t)(g - a.in[q].blk0) * P);
        }
        __syncthreads();
        {
            float *stale = state ? I.work + (size_t)(c - 2) * p + e0 : nullptr;
            if (N == 16) rounds<16, P>(sm, WS, 16, c, w, lane, stale, a.ld_w, P);
            else rounds<0, P>(sm, WS, N, c, w, lane, stale, a.ld_w, P);
        }
        __syncthreads();
        // decode: ghat_w = Y_w R_w
        v4f dacc[MTC][2];
#pragma unroll
        for (int mt = 0; mt < MTC; ++mt) dacc[mt][0] = dacc[mt][1] = v4f{0.f, 0.f, 0.f, 0.f};
        auto column = [&](int kk) {                       // Y column kk at this lane's positions
            const float *row = mine + (kk - (N - 1) + (kk < N - 1 ? K : 0)) * P + 2 * col;
            return kk < K ? *reinterpret_cast<const v2f *>(row) : kNoRow;
        };
        SplitRange range;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            const int k0 = 32 * kc + 8 * (int)opaque((uint32_t)g4);
            v2f y[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                y[s] = column(min(k0 + s, K));
                range.add(y[s]);
            }
            const Split3<v8bf> b0 = split8([&](int s) { return y[s][0]; }), b1 = split8([&](int s) { return y[s][1]; });
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt) {
                const Split3<v8bf> A = global_a32(dt + (size_t)mt * TD, kc, opaque(lane));
                dacc[mt][0] = mma_split32(A, b0, dacc[mt][0]);
                dacc[mt][1] = mma_split32(A, b1, dacc[mt][1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (K > 32 * KC) {
            const int k0 = 32 * KC + 4 * (int)opaque((uint32_t)g4);
            v2f y[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                y[s] = column(min(k0 + s, K));
                range.add(y[s]);
            }
            const Split3<v4bf> b0 = split4([&](int s) { return y[s][0]; }), b1 = split4([&](int s) { return y[s][1]; });
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt) {
                const Split3<v4bf> A = global_a16(dt + (size_t)mt * TD, KC, lane);
                dacc[mt][0] = mma_split16(A, b0, dacc[mt][0]);
                dacc[mt][1] = mma_split16(A, b1, dacc[mt][1]);
            }
        }
        const Contract how = range.contract(a.coefs, [&](auto f) __attribute__((always_inline)) {
#pragma unroll 1
            for (int kk = (int)opaque((uint32_t)g4); kk < K; kk += 4) f(column(kk));
        });
        if (how != kUsual)
            tiles_f32(dacc, MT, a.dfrag + (size_t)w * MT * a.KSd * 64, a.KSd, (int)opaque((uint32_t)lane),
                      [&](int k, int t) { return column(min(k, K))[t]; });
        // the observations to their slots (see k_ring_pass), four rows at a time
        if (state) {
            float *own = I.work + (size_t)w * a.ld_w + (size_t)(c - 1) * p + e0;
            float *rcv = I.work + (size_t)pv * a.ld_w + e0;
            float *pool = I.pool + (size_t)pv * N * ps + e0;
            const bool narrow = p < kNarrow;
            const uint32_t lane_row = opaque((uint32_t)(((size_t)g4 * p + 2 * (size_t)col) * sizeof(float)));
            float *row4 = step(rcv, (size_t)0) - (size_t)N * p;   // column 4 ks, for 4 ks >= N
            const float *yin = mine + (g4 - (N - 1)) * P + 2 * col;
#pragma unroll 4
            for (int ks = 0; 4 * ks < K; ++ks) {
                if (narrow && 4 * ks >= N && 4 * ks + 3 < K - 1) {
                    gstore<2>(row4, lane_row, *reinterpret_cast<const v2f *>(yin + 4 * ks * P));
                } else {
                    const int kk = 4 * ks + (int)opaque((uint32_t)g4);
                    if (kk < K)
                        gstore<2>((kk < N ? pool + (size_t)kk * ps : (kk < K - 1 ? rcv + (size_t)(kk - N) * p : own)) + 2 * col,
                                  0, column(kk));
                }
                row4 = step(row4, 4 * p);
            }
        }
        float *out = I.out + (size_t)w * a.ld_o;
        if (p < kNarrow && (size_t)(c - 1) * p + e0 + P <= d) {
            const uint32_t lane_out = opaque((uint32_t)(((size_t)(4 * g4) * p + 2 * (size_t)col) * sizeof(float)));
            float *row = out + e0;
            const bool ragged = a.ragged;
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt) {
                const int lrow = EXC ? 0 : 4 * (int)opaque((uint32_t)g4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const v2f v = {dacc[mt][0][r], dacc[mt][1][r]};
                    if (EXC || 16 * mt + lrow + r < c) {
                        if (ragged) gstore_cached<2>(row, lane_out, v);
                        else gstore<2>(row, lane_out, v);
                    }
                    row = step(row, r < 3 ? p : 13 * p);
                }
            }
        } else {
            const size_t pq = opaque_s(p);
            const int lrow = 4 * (int)opaque((uint32_t)g4), lcol = 2 * (int)opaque((uint32_t)col);
#pragma unroll
            for (int mt = 0; mt < MTC; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + lrow + r;
                    const size_t flat = (size_t)m * pq + e0 + lcol;
                    if (m < c && flat + 1 < d) gstore<2>(out + flat, 0, v2f{dacc[mt][0][r], dacc[mt][1][r]});
                    else if (m < c && flat < d) gstore1(out + flat, dacc[mt][0][r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        if (!more) break;
        encode(a.in[q], (size_t)(g - a.in[q].blk0) * P);  // reads and writes this wave's own rows only
    }
}

// All rounds of Algorithm 1 in one launch, where the call does not go in one
// pass: encoded chunks from `work`, observations to their slots.  N
// waves; each loads its worker's chunk rows (four rows of 64 positions per
// instruction) and stores the observations of the worker it receives for.
//
// Streams rows through LDS in groups of R rounds: a region of N + R rows per
// worker holds the chunks of the last N rounds (still to be subtracted) and
// of the group; the observation of round k takes the row of chunk k - N, is
// stored after the group, and the group after next loads into it.
//
// Bound by memory: reads every chunk and writes every observation once (2c + N
// rows per worker) where one launch per round moves 4c + 2N.  N = 16, c = 128,
// d = 1e8: 4.78 -> 3.03 ms (4.5 TB/s).  Groups of 16 rounds: one load of four
// rows per wave and K-quad, and at N = 16 the 32 rows of 64 positions fill 128 of
// the 160 KB of LDS.
constexpr int kGroup = 16;

template <int NX>
__device__ __forceinline__ void group_rounds(float *rows, int WS, int N, int c, int wave, int lane0, int k0, int k1,
                                             float (&x)[2]) {
    constexpr int P = 64;
    const int lane = (int)opaque((uint32_t)lane0);
    const int PW = NX ? 64 / (NX ? NX : 1) : 64 / N;
    const int rw = NX ? lane % (NX ? NX : 1) : lane / PW, rp = NX ? lane / (NX ? NX : 1) : lane - rw * PW;
    const int prev_addr = NX ? 0 : 4 * (rw == 0 ? lane + (N - 1) * PW : lane - PW);
    const bool first = rw == 0;
    const int C = N + kGroup;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int pos = (wave + h * N) * PW + rp;
        if ((wave + h * N) * PW >= P) break;
        if (rw >= N || pos >= P) continue;                // whole positions drop out: all N lanes of one
        float *S = rows + rw * WS + pos;
        int k = k0;
        if (k == 0) {
            x[h] = S[0];                                  // x_{rw,1} = delta_{rw,1}
            k = 1;
        }
        int sa = k % C, sy = (k + kGroup) % C;            // rows of chunk k and of chunk k - N
        for (; k < k1; ++k) {
            const float add = S[sa * P], sub = S[sy * P];
            const float recv = from_prev<NX>(x[h], prev_addr, first);
            S[sy * P] = recv;
            if (k < N) x[h] = recv + add;
            else if (k < c) x[h] = combine3(recv, sub, add);
            else x[h] = recv - sub;
            sa = sa + 1 == C ? 0 : sa + 1;
            sy = sy + 1 == C ? 0 : sy + 1;
        }
    }
}

__global__ __launch_bounds__(1024) void k_rounds_pass(PassParams a) {
    typedef Vec<4>::T VT;
    constexpr int P = 64, R = kGroup, Q = R / 4;
    extern __shared__ __align__(16) float sm[];
    const int N = a.N, c = a.c, K = c + N - 1, C = N + R;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, krow = lane >> 4;
    const int WS = pass_region(N, C, P);
    const int pv = w == 0 ? N - 1 : w - 1;                // the worker whose messages w receives
    float *mine = sm + w * WS + 4 * col;
    int q = 0;
    const Sweep sw = sweep_of(a);
    for (unsigned g = sw.first; g < sw.end; g += sw.step) {
        while (q + 1 < a.n && a.in[q + 1].blk0 <= g) ++q;
        const PassInst &I = a.in[q];
        const size_t p = I.p, ps = I.pool_stride;
        const size_t e = (size_t)(g - I.blk0) * P + 4 * col;
        const bool in = e < p;                            // p is a multiple of 32: a lane's four positions are in or out
        const float *src = I.work + (size_t)w * a.ld_w + e;
        float *rcv = I.work + (size_t)pv * a.ld_w + e;
        float *pool = I.pool + (size_t)pv * N * ps + e;
        VT b[Q];
        auto load = [&](int r0) {                         // chunks r0 .. r0 + R - 1 of worker w
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                const int r = r0 + 4 * u + krow;
                b[u] = (VT)0.f;
                if (in && r < c) b[u] = gload<4>(src + (size_t)r * p, 0);
            }
        };
        auto put = [&](int r0) {
#pragma unroll
            for (int u = 0; u < Q; ++u) *reinterpret_cast<VT *>(mine + (r0 + 4 * u + krow) % C * P) = b[u];
        };
        float x[2] = {0.f, 0.f};
        __syncthreads();                                  // the block before is out of LDS
        load(0);
        put(0);
        load(R);
        for (int k0 = 0; k0 < K; k0 += R) {
            const int k1 = min(K, k0 + R);
            __syncthreads();
            if (N == 8) group_rounds<8>(sm, WS, 8, c, w, lane, k0, k1, x);
            else if (N == 4) group_rounds<4>(sm, WS, 4, c, w, lane, k0, k1, x);
            else if (N == 2) group_rounds<2>(sm, WS, 2, c, w, lane, k0, k1, x);
            else if (N == 16) group_rounds<16>(sm, WS, 16, c, w, lane, k0, k1, x);
            else group_rounds<0>(sm, WS, N, c, w, lane, k0, k1, x);
            __syncthreads();
            // round k's observation is column k - 1 of Y_w: message k of worker pv
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                const int k = k0 + 4 * u + krow;
                const VT y = *reinterpret_cast<const VT *>(mine + (k + R) % C * P);
                if (in && k >= 1 && k < k1)
                    gstore<4>(k <= N ? pool + (size_t)(k - 1) * ps : rcv + (size_t)(k - 1 - N) * p, 0, y);
            }
            if (k0 + R < K) {
                put(k0 + R);
                load(k0 + 2 * R);
            }
        }
    }
}

// A kernel that takes PassParams, its LDS and its launch size.
struct PassKernel {
    void (*fn)(PassParams);
    size_t lds;
    int sweeps;
};

template <int MTC, int KSD, int V, int MAXT, int WPE>
PassKernel one_pass(int N, int c, int sweeps) {
    return {c == 16 * MTC ? k_ring_pass<MTC, KSD, V, true, MAXT, WPE> : k_ring_pass<MTC, KSD, V, false, MAXT, WPE>,
            pass_lds(N, c, V), sweeps};
}

// sweeps: workgroups per one that the chip holds at a time.  More of them
// level the end of the launch and keep the resident ones out of step; each
// loads its coefficients and its first block with nothing to hide behind.
// Many pay while the coefficients are few (16 against 1: N = 8, c = 16 379
// against 392 us, N = 4, c = 12 575 against 606; 8 against 1: N = 8, c = 32 2.66
// against 2.68 ms), one is best beyond (1 against 8: N = 2, c = 48 319 against 345
// us, N = 8, c = 48 1.63 against 1.66 ms, N = 4, c = 64 827 against 867 us, N = 16,
// c = 32 2.08 against 2.14 ms).
PassKernel ring_kernel(int N, int c) {
    if (N > 8) {
        if (c <= 16) return one_pass<1, 8, 2, 1024, 4>(N, c, 16);
        if (c <= 32) return one_pass<2, 12, 2, 1024, 4>(N, c, 1);
        return {c < 64 ? k_ring_pass_split<false> : k_ring_pass_split<true>, pass_lds(N, c, 2), 1};
    }
    switch ((c + 15) / 16) {
        case 1: return one_pass<1, 6, 4, 512, 4>(N, c, 16);
        case 2: return one_pass<2, 10, 4, 512, 4>(N, c, 8);
        case 3: return one_pass<3, 14, 2, 512, 2>(N, c, 1);
        default: return one_pass<4, 18, 2, 512, 2>(N, c, 1);
    }
}

PassKernel rounds_kernel(int N) {
    return {k_rounds_pass, (size_t)N * pass_region(N, N + kGroup, 64) * sizeof(float), 4};
}

// Workgroups of N waves that one CU holds at a time: what the LDS and the
// kernel's own registers (512 per lane and SIMD, in eights) allow.
hipError_t per_cu(const PassKernel &k, int N, int *wgs) {
    hipFuncAttributes at;
    const hipError_t e = hipFuncGetAttributes(&at, reinterpret_cast<const void *>(k.fn));
    if (e != hipSuccess) return e;
    const int waves = std::min(8, 512 / std::max(8, (at.numRegs + 7) / 8 * 8));
    *wgs = std::max(1, std::min((int)(kPassLds / k.lds), 4 * waves / N));
    return hipSuccess;
}

void start(const PassKernel &k, const PassParams &a, int cus, int wgs_per_cu, hipStream_t s) {
    const unsigned blocks = a.ragged ? (a.nblk + 7) / 8 * 8 : a.nblk;
    const unsigned wgs = std::min<unsigned>(blocks, (unsigned)(cus * wgs_per_cu * k.sweeps));
    hipLaunchKernelGGL(k.fn, dim3(wgs), dim3(64u * (unsigned)a.N), k.lds, s, a);
}

}  // namespace

// N <= 16, c <= 64 (K = c + N - 1 <= 80 there, one split tail): beyond that a
// block of all workers' rows does not fit the LDS, or the coefficients' way
// through the L2 outgrows the gradient's through memory.
int pass_positions(int N, int c) {
    if (N > 16 || c > 64) return 0;
    return N <= 8 && c <= 32 ? 64 : 32;
}

int rounds_positions(int N) { return N <= 16 ? 64 : 0; }

hipError_t prepare_passes(int N, int c, PassSize *out) {
    hipError_t e = hipSuccess;
    if (pass_positions(N, c)) e = per_cu(ring_kernel(N, c), N, &out->ring);
    if (e == hipSuccess && rounds_positions(N)) e = per_cu(rounds_kernel(N), N, &out->rounds);
    return e;
}

void launch_rounds_pass(const PassParams &a, int cus, const PassSize &size, hipStream_t s) {
    start(rounds_kernel(a.N), a, cus, size.rounds, s);
}

void launch_ring_pass(const PassParams &a, int cus, const PassSize &size, hipStream_t s) {
    start(ring_kernel(a.N, a.c), a, cus, size.ring, s);
}

}  // namespace cerar
