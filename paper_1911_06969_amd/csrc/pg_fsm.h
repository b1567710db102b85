// Numbering of labelled patterns (the dense index of the public header),
// shared by the two FSM pipelines.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pg {

// ----------------------------------------------------- pattern numbering

struct PatBase {
    int64_t L;
    int64_t p2, t3, paths;
    int64_t edge, wedge, tri, path, star;
    // four edges: 5-path, 4-star, fork, 4-cycle, paw
    int64_t q4, s4n, p5n, fkn, c4n, pwn;
    int64_t p5, star4, fork, cyc, paw;
    int64_t total;
};

__host__ __device__ inline PatBase pat_base(int64_t L, int max_edges) {
    PatBase B;
    B.L = L;
    B.p2 = L * (L + 1) / 2;
    B.t3 = L * (L + 1) * (L + 2) / 6;
    B.paths = (L * L * L * L + L * L) / 2;
    B.edge = 0;
    B.wedge = B.p2;
    B.tri = B.wedge + L * B.p2;
    B.path = B.tri + B.t3;
    B.star = B.path + B.paths;
    // label multisets of four leaves; palindromic 5-sequences; cycles up to
    // rotation and reflection (Burnside over the 8 symmetries of a square)
    B.q4 = L * (L + 1) * (L + 2) * (L + 3) / 24;
    B.p5n = (L * L * L * L * L + L * L * L) / 2;
    B.s4n = L * B.q4;
    B.fkn = L * B.p2 * L * L;
    B.c4n = (L * L * L * L + 2 * L * L * L + 3 * L * L + 2 * L) / 8;
    B.pwn = L * L * B.p2;
    B.p5 = B.star + L * B.t3;
    B.star4 = B.p5 + B.p5n;
    B.fork = B.star4 + B.s4n;
    B.cyc = B.fork + B.fkn;
    B.paw = B.cyc + B.c4n;
    B.total = max_edges >= 4 ? B.paw + B.pwn
              : max_edges == 3 ? B.p5 : (max_edges == 2 ? B.tri : B.p2);
    return B;
}

// rank of a <= b among label pairs in lexicographic order
__host__ __device__ inline int64_t pair_rank(int64_t a, int64_t b, int64_t L) {
    return a * L - a * (a - 1) / 2 + (b - a);
}

// rank of a <= b <= c among sorted label triples in lexicographic order
__host__ __device__ inline int64_t triple_rank(int64_t a, int64_t b, int64_t c, int64_t L) {
    int64_t r = 0;
    for (int64_t x = 0; x < a; ++x) r += (L - x) * (L - x + 1) / 2;
    for (int64_t y = a; y < b; ++y) r += L - y;
    return r + (c - b);
}

}  // namespace pg
