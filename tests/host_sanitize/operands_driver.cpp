// Prints which operand sets the plan builder prepares, per (N, c): the fp32
// fragments and the split ones of the encode and the decode, in elements.
#include <cstdio>
#include <vector>
#include "cerar.h"
#include "cerar_internal.hpp"
namespace cerar { void release_device(cerar_plan *) {} }

int main() {
    for (int N : {2, 8, 9, 16, 17, 18, 24, 40})
        for (int c : {16, 32, 33, 40, 47, 48, 50, 63, 64, 65, 96, 97, 128}) {
            if (c < N) continue;
            cerar_plan p;
            p.N = N;
            p.c = c;
            p.L = c + N - 2;
            p.U.assign((size_t)N * c * c, 0.5);
            p.R.assign((size_t)N * (c + N - 1) * c, 0.5);
            cerar::build_fragments(&p);
            std::printf("%d %d %d %zu %zu %zu %zu\n", N, c, p.KC, p.enc_frag.size(), p.dec_frag.size(),
                        p.enc_split.size(), p.dec_split.size());
        }
    return 0;
}
