// 5-motifs of graphs whose degrees are at most 64, from sums over vertices.
//
// A copy of a connected 5-vertex graph H (not necessarily induced) is counted from
// what one vertex a, its neighbours and the ends of the two-step paths from it
// know: degrees, the numbers of common neighbours c(a, w), the rows R of the graph
// on a's neighbours, and the closed walks of five steps.  The 21 sums are
//   trees                from degrees, less closed cases (triangles, 4-cycles);
//   5-cycles             closed 5-walks, less those on triangles and triangles with
//                        a tail;
//   4-cycle patterns     from c(a, w): with a tail, with a triangle on an edge,
//                        K2,3 (and with an edge among the three);
//   triangle patterns    from row sizes at either end of an edge;
//   patterns with a vertex adjacent to the other four: copies of the 4-vertex
//                        rest among a's neighbours (paths, paws, 4-cycles,
//                        diamonds, K4: gem, K4 and a vertex on two of its, wheel, K5
//                        less an edge, K5).
// A denser graph holds a fixed number of copies of a sparser one, so the induced
// counts follow from the densest down.
//
// The walk over all induced 5-sets that this takes the place of tests every
// extension of 25 million 4-sets against four lists; here a vertex costs its
// two-step paths, which fill a hash table in LDS, and one lookup per three-step
// path.  Uniform random graph, 100,000 vertices of 8 neighbours: 16.2 -> 0.52 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

namespace {

constexpr int M5_DEG = WAVE;         // a neighbour per lane, a row per 64-bit word
constexpr int M5_PATHS[2] = {320, M5_DEG * M5_DEG};   // two-step paths of a vertex per class of table
constexpr int M5_SLOTS[2] = {512, 8192};              // its entries: paths + neighbours + 1 at most three quarters
constexpr int M5_SUMS = 27;
constexpr int M5_STRIDE = 32;        // sums per copy (several copies: see STAT_COPIES)

enum Sum {
    S_STAR, S_FORK, S_PATH, S_DT, S_TRI, S_C4, S_CRICKET, S_BULL, S_LOLLI, S_DIAMOND, S_BANNER, S_WALK5, S_TAIL,
    S_BUTTERFLY, S_HOUSE, S_DART, S_KITE, S_K23, S_K4P, S_K4, S_BOOK, S_GEM, S_K5P3, S_K5E, S_W4, S_K5, S_K23E
};

constexpr uint32_t NO_KEY = ~0u;     // ids are below 2^31

template <int CLS>
struct M5Lds {
    uint32_t key[M5_SLOTS[CLS]];
    uint32_t val[M5_SLOTS[CLS]];     // c(a, key) | (place among a's neighbours + 1) << 16
    uint32_t path[M5_PATHS[CLS]];    // ends of the two-step paths
    uint16_t slot[M5_PATHS[CLS]];    // their table entries
    uint8_t from[M5_PATHS[CLS]];     // their middle vertices' places
    unsigned long long row[M5_DEG];
    int32_t deg[M5_DEG], pre[M5_DEG];
    int64_t start[M5_DEG];
};

// entry of key k, or (FIND) -1; otherwise it is made
template <int CLS, bool FIND>
__device__ __forceinline__ int m5_entry(uint32_t* key, uint32_t k) {
    constexpr uint32_t mask = M5_SLOTS[CLS] - 1;
    uint32_t h = (k * 0x9E3779B1u) >> (32 - (CLS == 0 ? 9 : 13));
    while (true) {
        uint32_t x = FIND ? key[h] : atomicCAS(&key[h], NO_KEY, k);
        if (x == k) return (int)h;
        if (x == NO_KEY) return FIND ? -1 : (int)h;
        h = (h + 1) & mask;   // ends: the table has empty entries
    }
}

__device__ __forceinline__ uint64_t choose2(uint64_t x) { return x * (x - 1) / 2; }   // x = 0: 0

__device__ __forceinline__ uint64_t choose3(uint64_t x) { return x < 3 ? 0 : x * (x - 1) * (x - 2) / 6; }

}  // namespace

// A wave per vertex.  CLS = 0 leaves the vertices of more than M5_PATHS[0] two-step
// paths to CLS = 1 (`more`, *n_more).  Bound by latency (a chain of six dependent loads a vertex) and by
// the lookups of the three-step paths, a list per lane.
template <int CLS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_motif5_sums(int64_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ col, int32_t* __restrict__ more,
                                                         uint32_t* __restrict__ n_more,
                                                         unsigned long long* __restrict__ out) {
    extern __shared__ unsigned long long shared[];   // an M5Lds per wave
    __shared__ unsigned long long total[M5_SUMS];
    const int w = threadIdx.x / WAVE;
    M5Lds<CLS>& L = reinterpret_cast<M5Lds<CLS>*>(shared)[w];
    if (threadIdx.x < M5_SUMS) total[threadIdx.x] = 0ull;
    for (int i = lane(); i < M5_SLOTS[CLS]; i += WAVE) {
        L.key[i] = NO_KEY;
        L.val[i] = 0u;
    }
    __syncthreads();
    uint64_t S[M5_SUMS];
#pragma unroll
    for (int i = 0; i < M5_SUMS; ++i) S[i] = 0;
    const int64_t waves = (int64_t)gridDim.x * (THREADS / WAVE);
    const int64_t items = CLS == 0 ? n : (int64_t)*n_more;
    for (int64_t it = (int64_t)blockIdx.x * (THREADS / WAVE) + w; it < items; it += waves) {
        const int64_t a = CLS == 0 ? it : (int64_t)uniform(more[it]);
        const int64_t r0 = uniform64(rp[a]);
        const int d = (int)(uniform64(rp[a + 1]) - r0);   // at most M5_DEG
        if (d == 0) continue;
        const bool on = lane() < d;
        int32_t u = 0, du = 0;
        int64_t su = 0;
        if (on) {
            u = col[r0 + lane()];
            su = rp[u];
            du = (int32_t)(rp[u + 1] - su);
        }
        const uint32_t inc = wave_incl_scan((uint32_t)du);
        const int np = (int)bcast(inc, WAVE - 1);   // two-step paths, back to a included
        if (CLS == 0 && np > M5_PATHS[0]) {
            if (lane() == 0) more[atomicAdd(n_more, 1u)] = (int32_t)a;
            continue;
        }
        wave_sync();   // the previous vertex's entries are cleared
        int own = 0;
        if (on) {
            L.start[lane()] = su;
            L.deg[lane()] = du;
            L.pre[lane()] = (int32_t)inc - du;
            L.row[lane()] = 0ull;
            own = m5_entry<CLS, false>(L.key, (uint32_t)u);
            L.val[own] = (uint32_t)(lane() + 1) << 16;
        }
        wave_sync();
        // two-step paths: counts per end, and the rows among the neighbours
        for (int k0 = 0; k0 < np; k0 += WAVE) {
            const int k = k0 + lane();
            if (k < np) {
                int lo = 0, hi = d - 1;   // the last list that starts at k or before
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (L.pre[mid] <= k) lo = mid; else hi = mid - 1;
                }
                const uint32_t x = (uint32_t)col[L.start[lo] + (k - L.pre[lo])];
                const int e = m5_entry<CLS, false>(L.key, x);
                const uint32_t at = atomicAdd(&L.val[e], 1u) >> 16;
                if (at) atomicOr(&L.row[lo], 1ull << (at - 1));
                L.path[k] = x;
                L.slot[k] = (uint16_t)e;
                L.from[k] = (uint8_t)lo;
            }
        }
        wave_sync();
        const uint64_t R = on ? L.row[lane()] : 0ull;
        const uint64_t t = (uint64_t)popc64(R);
        const uint64_t D = (uint64_t)d, dn = (uint64_t)du;
        const uint64_t ta = wave_sum_u32((uint32_t)t) / 2;   // triangles at a
        const uint64_t s1 = (uint64_t)(np - d);              // sum of the neighbours' degrees less one
        if (on) {
            S[S_FORK] += (dn - 1) * choose2(D - 1) - t * (D - 2);
            S[S_PATH] -= (dn - 1) * (dn - 1);
            S[S_DT] += t * D;
            S[S_TRI] += t;
            S[S_CRICKET] += t ? t * choose2(D - 2) : 0;
            S[S_BULL] += t * (D - 2) * (dn - 2) - t * (t - 1);
            S[S_LOLLI] += (ta - t) * (dn - 1);
            S[S_DIAMOND] += choose2(t);
            S[S_TAIL] += t * (D - 2);
            S[S_DART] += choose2(t) * (D + dn - 6);
            S[S_BOOK] += choose3(t);
        }
        if (lane() == 0) {
            S[S_STAR] += d < 4 ? 0 : D * (D - 1) * (D - 2) * (D - 3) / 24;
            S[S_PATH] += s1 * s1;
            S[S_BUTTERFLY] += choose2(ta);
        }
        for (int k = lane(); k < np; k += WAVE) {
            const uint32_t x = L.path[k];
            const uint64_t c = L.val[L.slot[k]] & 0xffffu;
            if (x != (uint32_t)a) {
                const int i = L.from[k];
                const uint64_t Ri = L.row[i];
                S[S_C4] += c - 1;
                S[S_BANNER] += (c - 1) * (D - 2);
                S[S_HOUSE] += (c - 1) * (uint64_t)popc64(Ri);
                S[S_K23] += (c - 1) * (c - 2);
                if (c > 2)   // K2,3 and an edge: x adjacent to two neighbours that are
                    for (uint64_t js = Ri; js; js &= js - 1) {
                        const int j = __builtin_ctzll(js);
                        if (contains(col + L.start[j], L.deg[j], (int32_t)x)) S[S_K23E] += c - 2;
                    }
            }
            // three-step paths: walks of two steps back to a
            const int64_t x0 = rp[x], x1 = rp[x + 1];
            for (int64_t y = x0; y < x1; ++y) {
                const int e = m5_entry<CLS, true>(L.key, (uint32_t)col[y]);
                if (e >= 0) S[S_WALK5] += L.val[e] & 0xffffu;
            }
        }
        if (ta > 0) {
            uint64_t cs = 0;
            for (uint64_t js = R; js; js &= js - 1) {
                const int j = __builtin_ctzll(js);
                const uint64_t Rj = L.row[j];
                const uint64_t c = (uint64_t)popc64(R & Rj);
                cs += c;
                S[S_KITE] += (t - 1) * (uint64_t)(L.deg[j] - 2);
                S[S_GEM] += (t - 1) * (uint64_t)(popc64(Rj) - 1);
                S[S_K5E] += choose2(c);
                if (c && j > lane())
                    for (uint64_t ls = R & Rj & (~0ull << j); ls; ls &= ls - 1)   // Rj has no bit j
                        S[S_K5] += (uint64_t)popc64(ls & (ls - 1) & L.row[__builtin_ctzll(ls)]);
            }
            S[S_K4] += cs;
            S[S_K4P] += cs * (D - 3);
            S[S_K5P3] += cs * (t - 2);
            for (int j = 0; j < d; ++j)
                if (lane() < j) S[S_W4] += choose2((uint64_t)popc64(R & L.row[j]));
        }
        wave_sync();
        for (int k = lane(); k < np; k += WAVE) {
            L.key[L.slot[k]] = NO_KEY;
            L.val[L.slot[k]] = 0u;
        }
        if (on) {
            L.key[own] = NO_KEY;
            L.val[own] = 0u;
        }
        wave_sync();
    }
#pragma unroll
    for (int i = 0; i < M5_SUMS; ++i) {
        const uint64_t x = wave_sum_u64(S[i]);
        if (lane() == 0 && x) atomicAdd(&total[i], (unsigned long long)x);
    }
    __syncthreads();
    if (threadIdx.x < M5_SUMS && total[threadIdx.x])
        atomicAdd(&out[(blockIdx.x % STAT_COPIES) * M5_STRIDE + threadIdx.x], total[threadIdx.x]);
}

template <int CLS, int THREADS>
static void launch_sums(pg_graph* g, int64_t items, int32_t* more, uint32_t* n_more, unsigned long long* out) {
    const auto kernel = k_motif5_sums<CLS, THREADS>;
    const size_t lds = sizeof(M5Lds<CLS>) * (THREADS / WAVE);
    if (lds > 64 * 1024)
        PG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
    const int64_t most = (items + THREADS / WAVE - 1) / (THREADS / WAVE);
    kernel<<<queue_blocks(kernel, THREADS, lds, most), THREADS, lds, g->stream>>>(
        g->n, g->rp.as<int64_t>(), g->col.as<int32_t>(), more, n_more, out);
    PG_HIP(hipGetLastError());
}

bool count_motifs5_sums(pg_graph* g, const Motif5Table& T, uint64_t* counts) {
    if (g->max_deg > M5_DEG) return false;
    hipStream_t s = g->stream;
    Arena& ar = g->arena;
    constexpr int words = STAT_COPIES * M5_STRIDE;
    uint64_t* small = push<uint64_t>(ar, words + 1);
    int32_t* more = push<int32_t>(ar, (size_t)std::max<int64_t>(g->n, 1));
    unsigned long long* out = reinterpret_cast<unsigned long long*>(small);
    uint32_t* n_more = reinterpret_cast<uint32_t*>(small + words);
    fill_u64(small, words + 1, 0, s);
    {
        ProfScope ps("motif_last", s, (double)g->n);
        launch_sums<0, 256>(g, g->n, more, n_more, out);
        if (g->max_deg * g->max_deg > M5_PATHS[0]) launch_sums<1, WAVE>(g, g->n, more, n_more, out);
    }
    uint64_t h[words], S[M5_STRIDE] = {};
    PG_HIP(hipMemcpyAsync(h, small, sizeof(h), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    for (int i = 0; i < words; ++i) S[i % M5_STRIDE] += h[i];
    // copies of the 21 graphs (each as one of its edge masks, bit b (b - 1) / 2 + a)
    const uint64_t triangles = S[S_TRI] / 6, c4 = S[S_C4] / 8, diamonds = S[S_DIAMOND] / 2, k4 = S[S_K4] / 24;
    auto edges = [](std::initializer_list<std::pair<int, int>> es) {
        int m = 0;
        for (auto [a, b] : es) m |= 1 << (b * (b - 1) / 2 + a);   // a < b
        return m;
    };
    struct Copies {
        int mask;
        uint64_t n;
    };
    const Copies copies[21] = {
        {edges({{0, 1}, {0, 2}, {0, 3}, {0, 4}}), S[S_STAR]},
        {edges({{0, 1}, {0, 2}, {0, 3}, {3, 4}}), S[S_FORK]},
        // pairs of two steps from the middle, less those that meet
        {edges({{0, 1}, {1, 2}, {2, 3}, {3, 4}}), S[S_PATH] / 2 - (S[S_DT] - 9 * triangles) - 4 * c4},
        // triangle and two tails: at one vertex, at two, one after the other
        {edges({{0, 1}, {0, 2}, {1, 2}, {0, 3}, {0, 4}}), S[S_CRICKET] / 2},
        {edges({{0, 1}, {0, 2}, {1, 2}, {0, 3}, {1, 4}}), S[S_BULL] / 2},
        {edges({{0, 1}, {0, 2}, {1, 2}, {0, 3}, {3, 4}}), S[S_LOLLI] - 4 * diamonds},
        // 4-cycle and a tail; 5-cycle
        {edges({{0, 1}, {1, 2}, {2, 3}, {0, 3}, {0, 4}}), S[S_BANNER] / 2 - 2 * diamonds},
        {edges({{0, 1}, {1, 2}, {2, 3}, {3, 4}, {0, 4}}), (S[S_WALK5] - 30 * triangles - 5 * S[S_TAIL]) / 10},
        // two triangles at a vertex; 4-cycle and a triangle on its edge
        {edges({{0, 1}, {0, 2}, {1, 2}, {0, 3}, {0, 4}, {3, 4}}), S[S_BUTTERFLY] - 2 * diamonds},
        {edges({{0, 1}, {1, 2}, {2, 3}, {0, 3}, {0, 4}, {1, 4}}), S[S_HOUSE] / 2 - 4 * diamonds},
        // diamond (0, 1 on two triangles) and a tail at 0, at 2
        {edges({{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {0, 4}}), S[S_DART] / 2},
        {edges({{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 4}}), S[S_KITE] / 2 - 12 * k4},
        // K2,3; with an edge among the three
        {edges({{0, 2}, {0, 3}, {0, 4}, {1, 2}, {1, 3}, {1, 4}}), S[S_K23] / 12},
        {edges({{0, 2}, {0, 3}, {0, 4}, {1, 2}, {1, 3}, {1, 4}, {2, 3}}), S[S_K23E] / 4},
        // K4 and a tail; three triangles on an edge
        {edges({{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}, {0, 4}}), S[S_K4P] / 6},
        {edges({{0, 1}, {0, 2}, {0, 3}, {0, 4}, {1, 2}, {1, 3}, {1, 4}}), S[S_BOOK] / 2},
        // a vertex (0) on a path of four, on a 4-cycle, on a triangle with a tail
        {edges({{0, 1}, {0, 2}, {0, 3}, {0, 4}, {1, 2}, {2, 3}, {3, 4}}), S[S_GEM] / 2 - 12 * k4},
        {edges({{0, 1}, {0, 2}, {0, 3}, {0, 4}, {1, 2}, {2, 3}, {3, 4}, {1, 4}}), S[S_W4] / 2},
        {edges({{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}, {0, 4}, {1, 4}}), S[S_K5P3] / 4},
        // K5 less an edge; K5
        {1023 & ~1, S[S_K5E] / 6},
        {1023, S[S_K5] / 5},
    };
    for (const Copies& c : copies) counts[T.cls[c.mask]] = c.n;
    for (int i = 20; i >= 0; --i)   // classes are in order of edges
        for (int j = i + 1; j < 21; ++j) counts[i] -= (uint64_t)T.copies[i][j] * counts[j];
    return true;
}

}  // namespace pg
