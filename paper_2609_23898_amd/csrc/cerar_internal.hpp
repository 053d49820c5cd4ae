// Internal structures shared by the host plan code and the HIP launchers.
#pragma once

#include <cstdint>
#include <exception>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/cerar.h"

namespace cerar {

// Build limits (validated by cerar_plan_create*).
constexpr int kMaxN = 64;
constexpr int kMaxC = 128;
constexpr int kMaxNodePerms = 4096;    // candidate H permutations per plan

// The MFMA operand tiling of encode/decode: 16 output rows per M-tile, 4
// reduction rows per K-step, 64 lanes per fragment.
constexpr int kTileM = 16;
constexpr int kTileK = 4;
constexpr int kLanes = 64;

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Chunk length p is ceil(d/c) rounded up to a multiple of this many floats
// (128 bytes); the zero padding of the last chunk absorbs the difference.
constexpr size_t kChunkAlign = 32;

// One round's per-worker slot operands: next message dst = recv - sub + add
// (sub/add = -1 when absent; dst = -1 when the round only relabels).
struct RoundOp {
    int recv, sub, add, dst;
};

// Slot-ownership bookkeeping of the handoff ring for given (N, c).
// Slot s < N*c is chunk s % c of worker s / c in `work`; slot s >= N*c is
// pool slot s - N*c of the workspace (N per worker).
struct RingTables {
    int N = 0, c = 0, L = 0;
    std::vector<int> enc_copy;       // N: pool slot that receives x_{i,1} = delta_{i,1}
    std::vector<RoundOp> rounds;     // (L+1) x N, entry k*N + i for round k (row 0 unused)
    std::vector<int> ycols;          // N x (L+1): slots of Y_i = [B_1..B_{N-1} | D_1..D_c]
    std::vector<int> state;          // (L+1) x N x (c+N): D (c), B (N-1), next message (1)
    int pool_slots() const { return N * N; }
};

// Whether the plan contracts on fp32 operands (else on split ones, see
// split.hpp): where the one-pass kernel's waves keep the coefficients in their
// registers, eight waves those of c <= 64 and sixteen those of c <= 32.  The step
// calls follow the one-pass kernel, so that both give the same bits.  Beyond
// N = 16 there is none; there the split pays where c is no multiple of 16 (N =
// 24, d = 200000 c: c = 40 encode 391 us and decode 505 against 566 and 541 on
// masked fp32 tiles), is even at c = 64 (516 and 664 against 521 and 668), and at c =
// 48 the step decode loses what the bucketed call wins (493 against 465 us, 17
// buckets 2.13 against 2.20 ms), so one rule holds for all.
inline bool contracts_fp32(int N, int c) { return c <= (N <= 8 ? 64 : 32); }
// Chunks of 32 K-steps of the split contraction, or 0 where the fp32 one stays:
// 2, 3 or 4 for the encode, and that many and a 16-step tail for the decode
// where its K = c + N - 1 observations fit them.
inline int split_chunks(int N, int c) { return contracts_fp32(N, c) ? 0 : (c <= 64 ? 2 : (c <= 96 ? 3 : 4)); }
// What a plan's coefficients allow on split operands: everything; no scaling of
// half-blocks with small entries (some are 2^40 or more); nothing (some are not
// the sum of their three terms).
enum SplitCoefs { kCoefsUsual, kCoefsLarge, kCoefsFp32 };
inline bool split_decode_fits(int N, int c) { return c + N - 1 <= 32 * split_chunks(N, c) + 16; }
// bf16 of one 16-row tile of a worker's split operands: per chunk and term 64
// lanes of 8, and for the decode per term 64 lanes of 4 of the tail.  A worker
// has 2 KC tiles (zero beyond c rows).
constexpr int split_tile_encode(int KC) { return KC * 3 * 64 * 8; }
constexpr int split_tile_decode(int KC) { return KC * 3 * 64 * 8 + 3 * 64 * 4; }

// Builds the tables and checks that no launch reads a slot another worker
// writes in the same launch.  Returns an empty string or a diagnostic.
std::string build_ring_tables(int N, int c, RingTables &t);

// Workgroups that one compute unit holds at a time, of the plan's one-pass and
// rounds kernels (0 where it has none).
struct PassSize {
    int ring = 0, rounds = 0;
};

struct DeviceCopy {
    float *enc_frag = nullptr;       // N x MT x KSe x 64 fp32 fragments of U_i
    float *dec_frag = nullptr;       // N x MT x KSd x 64 fp32 fragments of R_i
    int *ycols = nullptr;            // N x (L+1) slot ids
    RoundOp *rounds = nullptr;       // (L+1) x N
    uint16_t *enc_split = nullptr;   // the split operands of U_i and R_i (plans with KC > 0)
    uint16_t *dec_split = nullptr;
    int cus = 0;                     // compute units of the device
    PassSize size;
};

}  // namespace cerar

struct cerar_plan {
    int N = 0, c = 0, L = 0;
    cerar_plan_info info{};
    std::vector<double> U;           // N x c x c: U[k][l][j]
    std::vector<double> R;           // N x (L+1) x c: R[i][k][m]
    std::vector<double> B, D;        // MPC base / perturbation (empty for EXPLICIT)
    int svd_sweeps = 80;             // cap on one-sided Jacobi sweeps per SVD (cerar_plan_desc.svd_sweeps)
    bool svd_ok = true;              // every SVD so far converged within svd_sweeps
    cerar::RingTables tab;
    int MT = 0, KSe = 0, KSd = 0;    // M-tiles, encode K-steps, decode K-steps
    std::vector<float> enc_frag, dec_frag;
    int KC = 0;                      // 32-step chunks of the split contraction, 0 where it is not used
    std::vector<uint16_t> enc_split, dec_split;   // bf16 bits, see split_tile_encode / split_tile_decode
    int split_coefs = 0;             // SplitCoefs of its coefficients
    mutable std::mutex dev_mu;
    mutable std::map<int, cerar::DeviceCopy> dev;   // per HIP device ordinal
};

namespace cerar {
// Thread-local error text; returns `status` for convenient `return fail(...)`.
int fail(int status, const char *fmt, ...) noexcept;
void clear_error() noexcept;

// Runs the body of a C entry point and turns a C++ exception into a status,
// so that none unwinds through the C ABI: a failed host allocation, or a
// host resource that could not be had, is CERAR_E_NOMEM.
template <class F>
int guarded(F &&body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail(CERAR_E_NOMEM, "out of host memory");
    } catch (const std::exception &e) {
        return fail(CERAR_E_NOMEM, "host resources exhausted: %s", e.what());
    } catch (...) {
        return fail(CERAR_E_NOMEM, "unexpected host exception");
    }
}

// Fills MT/KSe/KSd and the fp32 fragment arrays from U and R.
void build_fragments(cerar_plan *plan);
// Releases device copies (called by cerar_plan_destroy; defined with the kernels).
void release_device(cerar_plan *plan);
}  // namespace cerar
