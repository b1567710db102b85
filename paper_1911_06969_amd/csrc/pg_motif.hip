// Vertex-induced motif counting for k = 5 by extension (Pangolin sections
// 2.2, 3.3 motif Listing, 4.2), and the dispatch over k (k = 3 and 4:
// pg_motif_sums.hip).
//
// Canonical test (isAutoCanonical for vertex extension).  An embedding is
// kept in one order only: the breadth-first order from its smallest
// vertex, neighbours of one vertex taken in increasing id.  With p(j) the
// position of v_j's first earlier neighbour, a sequence is canonical iff
// v0 is the minimum, p is non-decreasing and p(j) = p(j+1) implies
// v_j < v_{j+1}.  Extending a canonical sequence by u is canonical iff
// u > v0, u is not in it, and with s = the first position adjacent to u:
// s >= p(last), and s = p(last) implies u > v_last.
//
// Levels.  L1 = every edge once as (v0 < v1) (p(1) = 0).  L2 = canonical
// connected 3-sets (v0, v1, v2) built by count / scan / write, each entry
// with a 2-bit connectivity code memoising its pattern (bit 0: v2 ~ v0,
// bit 1: v2 ~ v1; section 4.2 memoisation).  Level 3 is queued in LDS and the
// last level is fused with classification and reduction.
//
// Output order: k = 3: wedge, triangle; k = 4: path, star, cycle, paw,
// diamond, 4-clique; k = 5: the 21 classes described at k_motif_last5.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

constexpr int MO_THREADS = 128;
constexpr int MO_WAVES = MO_THREADS / WAVE;
constexpr int MO_STAGE = 512;     // adjacency lists up to this long are staged in LDS
constexpr int MO5_WAVES_PER_CU = 32;   // k = 5 last level: at most this many waves per CU (latency-bound lanes)

enum { ML1_COUNT = 0, ML1_WRITE = 1 };

struct MotifArgs {
    XcdQueue Q;                 // over items[]: (segment, round of 64 children)
    const uint64_t* items;
    const int64_t* rp;          // undirected CSR
    const int32_t* col;
    // level-1 segments: vertex v0 owns L1 entries l1_seg[v0] .. l1_seg[v0+1]-1
    const int64_t* l1_seg;
    const int32_t* l1_src;
    const int32_t* l1_dst;
    int64_t x_lo, x_hi;         // L1 entries extended
    uint32_t* count;            // ML1_COUNT: L2 children per L1 entry (indexed by entry)
    const uint64_t* start;      // ML1_WRITE: children of entry x at start[x] - start_base
    uint64_t start_base;
    int32_t* out_vid;
    uint8_t* out_code;
    // last level: segment p (an L1 entry) owns the L2 entries
    // seg2[p] - seg2_base .. seg2[p+1] - seg2_base - 1
    const uint64_t* seg2;
    uint64_t seg2_base;
    const int32_t* vid2;
    const uint8_t* code2;
    unsigned long long* out;    // pattern counters + work stats
    // dense rows of high-degree vertices: hub_id[v] >= 0 selects row
    // hub_bits + hub_id[v] * hub_words (bit u set iff u ~ v)
    const int32_t* hub_id;
    const uint32_t* hub_bits;
    int64_t hub_words;
};

// --------------------------------------------------------------- helpers

template <class P>
__device__ __forceinline__ bool member(P a, int32_t len, int32_t key) {
    return contains(a, len, key);
}

__device__ __forceinline__ const uint32_t* hub_row(const MotifArgs& A, int32_t v) {
    const int32_t h = A.hub_id[v];
    return h >= 0 ? A.hub_bits + (int64_t)h * A.hub_words : nullptr;
}

__device__ __forceinline__ bool bit_has(const uint32_t* row, int32_t u) {
    return (row[(uint32_t)u >> 5] >> (u & 31)) & 1u;
}

// membership in a sorted list, through its dense row when it has one
template <class P>
__device__ __forceinline__ bool adj_has(const uint32_t* row, P a, int32_t len, int32_t u) {
    return row ? bit_has(row, u) : member(a, len, u);
}

// relative cost of one membership test: 1 through LDS or a dense row,
// otherwise the depth of a binary search in global memory
__device__ __forceinline__ int32_t probe_cost(bool cheap, int32_t len) {
    return cheap ? 1 : 32 - __clz(max(len, 1));
}

// ---------------------------------------------------------- level 1 -> 2

struct L1Lds {
    int32_t A0[MO_WAVES][MO_STAGE];
    uint32_t pre[MO_WAVES][WAVE];
    int64_t lo1[MO_WAVES][WAVE];    // first entry of A1 above v0 (global index)
    int32_t d1[MO_WAVES][WAVE];     // |A1 above v0|
    int32_t v1[MO_WAVES][WAVE];
    int32_t na[MO_WAVES][WAVE];     // |A0 above v1|
    int32_t opt[MO_WAVES][WAVE];    // COUNT: 0 iterate A0', 1 iterate A1'
    int32_t hb1[MO_WAVES][WAVE];    // dense row of v1, or -1
    uint32_t c_all[MO_WAVES][WAVE];
};

// L1 entries [xc, x1) of vertex v0 (at most 64: one work item)
template <int MODE, class P0>
__device__ __forceinline__ void motif_l1_segment(const MotifArgs& A, L1Lds& L, int w, int32_t v0, P0 A0,
                                                 int32_t d0, int64_t r0, int64_t b, int32_t xc, int32_t x1,
                                                 const uint32_t* h0, bool a0_cheap) {
    // A0' = A0 above v0, at positions [a0lo, d0)
    const int32_t a0lo = (int32_t)upper_bound(A0, 0, d0, v0);
    {
        const int32_t x = xc + lane();
        uint32_t work = 0;
        if (x < x1) {
            const int32_t v1 = A.l1_dst[b + x];
            const int64_t q0 = A.rp[v1], q1 = A.rp[v1 + 1];
            const int64_t lo1 = upper_bound(A.col, q0, q1, v0);
            const int32_t d1p = (int32_t)(q1 - lo1);
            const int32_t na = d0 - (int32_t)upper_bound(A0, a0lo, d0, v1);
            const int32_t d0p = d0 - a0lo;
            const int32_t hb1 = A.hub_id[v1];
            int opt = 0;
            if (MODE == ML1_WRITE) {
                work = (uint32_t)(na + d1p);
            } else {
                // iterate A0' probing A1, or A1' probing A0: the cheaper total
                const int64_t c0 = (int64_t)d0p * probe_cost(hb1 >= 0, (int32_t)(q1 - q0));
                const int64_t c1 = (int64_t)d1p * probe_cost(a0_cheap, d0);
                opt = (c0 <= c1) ? 0 : 1;
                work = (uint32_t)(opt == 0 ? d0p : d1p);
            }
            L.lo1[w][lane()] = lo1;
            L.d1[w][lane()] = d1p;
            L.v1[w][lane()] = v1;
            L.na[w][lane()] = na;
            L.opt[w][lane()] = opt;
            L.hb1[w][lane()] = hb1;
        }
        const uint32_t inc = wave_incl_scan(work);
        const uint32_t W = bcast(inc, WAVE - 1);
        L.pre[w][lane()] = inc - work;
        L.c_all[w][lane()] = 0;
        wave_sync();
        const int nx = min(WAVE, x1 - xc);
        for (uint32_t t0 = 0; t0 < W; t0 += WAVE) {
            const uint32_t t = t0 + lane();
            const bool valid = t < W;
            int xi = 0;
            {
                int n_i = nx;
                while (n_i > 1) {
                    const int half = n_i >> 1;
                    if (L.pre[w][xi + half] <= t) xi += half;
                    n_i -= half;
                }
            }
            if (MODE != ML1_WRITE) {
                if (valid) {
                    const uint32_t j = t - L.pre[w][xi];
                    const int32_t v1 = L.v1[w][xi];
                    const int32_t hb1 = L.hb1[w][xi];
                    int32_t u;
                    bool f;
                    if (L.opt[w][xi] == 0) {
                        u = A0[a0lo + j];
                        if (hb1 >= 0) {
                            f = bit_has(A.hub_bits + (int64_t)hb1 * A.hub_words, u);
                        } else {
                            const int64_t q0 = A.rp[v1], q1 = A.rp[v1 + 1];
                            f = member(A.col + q0, (int32_t)(q1 - q0), u);
                        }
                    } else {
                        u = A.col[L.lo1[w][xi] + j];
                        f = adj_has(h0, A0, d0, u);
                    }
                    if (f) atomicAdd(&L.c_all[w][xi], 1u);
                }
            } else {
                // children of (v0, v1): u in A0 above v1 (code bit 0 set, bit 1 =
                // u ~ v1), then u in A1 above v0 not adjacent to v0 (code 2)
                bool emit = false;
                int32_t u = 0;
                uint8_t code = 0;
                if (valid) {
                    const uint32_t j = t - L.pre[w][xi];
                    const int32_t v1 = L.v1[w][xi];
                    const int32_t na = L.na[w][xi];
                    const int32_t hb1 = L.hb1[w][xi];
                    if ((int32_t)j < na) {
                        u = A0[d0 - na + (int32_t)j];
                        bool a12 = false;
                        if (hb1 >= 0) {
                            a12 = bit_has(A.hub_bits + (int64_t)hb1 * A.hub_words, u);
                        } else {
                            const int64_t q0 = A.rp[v1], q1 = A.rp[v1 + 1];
                            a12 = member(A.col + q0, (int32_t)(q1 - q0), u);
                        }
                        code = 1 | (a12 ? 2 : 0);
                        emit = true;
                    } else {
                        u = A.col[L.lo1[w][xi] + (j - (uint32_t)na)];
                        emit = !adj_has(h0, A0, d0, u);
                        code = 2;
                    }
                }
                const int key = valid ? xi : WAVE;
                const int prev = __shfl_up(key, 1, WAVE);
                const bool head = lane() == 0 || prev != key;
                const uint64_t H = ballot(head);
                const uint64_t F = ballot(emit);
                const uint64_t le = lanemask_lt() | (1ull << lane());
                const int h = 63 - __clzll(H & le);
                const uint64_t grp = le & ~((1ull << h) - 1ull);
                const uint32_t base = valid ? L.c_all[w][xi] : 0u;
                if (emit) {
                    const uint64_t dst = A.start[b + xc + xi] - A.start_base + base +
                                         (uint64_t)popc64(F & grp & lanemask_lt());
                    A.out_vid[dst] = u;
                    A.out_code[dst] = code;
                }
                const bool next_head = (lane() == WAVE - 1) || ((H >> (lane() + 1)) & 1ull);
                wave_sync();
                if (valid && next_head) L.c_all[w][xi] = base + (uint32_t)popc64(F & grp);
                wave_sync();
            }
        }
        wave_sync();
        if (x < x1) {
            if (MODE == ML1_COUNT) A.count[b + x] = (uint32_t)(L.na[w][lane()] + L.d1[w][lane()]) - L.c_all[w][lane()];
        }
        wave_sync();
    }
}

template <int MODE>
__global__ __launch_bounds__(MO_THREADS) void k_motif_l1(MotifArgs A) {
    __shared__ L1Lds L;
    const int w = threadIdx.x / WAVE;
    QueueCursor cur = queue_start();
    int64_t it_end = 0;
    for (int64_t it = queue_next(A.Q, cur, it_end); it >= 0; it = queue_next(A.Q, cur, it_end)) {
        for (int64_t j = it; j < it_end; ++j) {
            const uint64_t item = A.items[j];
            const int64_t p = item_seg(item);
            const int32_t v0 = (int32_t)p;
            const int64_t b = A.l1_seg[p], e = A.l1_seg[p + 1];
            const int32_t s = (int32_t)(e - b);
            // this item's entries, within the launch's window [x_lo, x_hi)
            const int32_t xa = (int32_t)max64(item_round(item) * WAVE, A.x_lo - b);
            const int32_t xb = (int32_t)min64(min64(item_round(item) * WAVE + WAVE, s), A.x_hi - b);
            if (xa >= xb) continue;
            const int64_t r0 = A.rp[v0], r1 = A.rp[v0 + 1];
            const int32_t d0 = (int32_t)(r1 - r0);
            if (d0 <= MO_STAGE) {
                for (int i = lane(); i < d0; i += WAVE) L.A0[w][i] = A.col[r0 + i];
                wave_sync();
                motif_l1_segment<MODE>(A, L, w, v0, &L.A0[w][0], d0, r0, b, xa, xb, nullptr, true);
            } else {
                const uint32_t* h0 = hub_row(A, v0);
                motif_l1_segment<MODE>(A, L, w, v0, A.col + r0, d0, r0, b, xa, xb, h0, h0 != nullptr);
            }
            wave_sync();
        }
    }
}

// ------------------------------------------------------- last level, k = 5
//
// (Graphs with a degree above 64: the others are counted from sums,
// pg_motif5.hip.)
//
// Five vertices: a pattern is the 10-bit mask of adjacent position pairs,
// bit b(b-1)/2 + a for a < b (the 4-vertex order followed by 04, 14, 24,
// 34).  Classes are the 21 connected graphs numbered by (edge count,
// smallest mask over the relabellings of the positions); the table maps a
// mask to its class (-1 when disconnected).
//
// Level 3 (four vertices) is not materialised.  A wave takes 64 L2 entries
// (v0, v1, v2) of one L1 entry (v0, v1), one per lane.  In rounds, every
// lane walks its entry's canonical extensions u by the rule above and
// queues each (v2, u, pair mask, p(3)) in the wave's LDS queue until the
// queue is full (a lane whose push does not fit retries that u in the next
// round); then the lanes take the queued 4-sets one each, walk their
// canonical extensions w and add one to the class of each 10-bit mask.  So
// lanes wait on the degrees of single 4-sets, not of whole subtrees.
// Adjacency is a binary search in the CSR.

constexpr int M5_Q = 512;       // queued 4-sets per wave
constexpr int M5_STAGE = 256;   // lists of v0 and v1 up to this long are staged in LDS

struct M5Lds {
    int32_t s0[MO_WAVES][M5_STAGE];
    int32_t s1[MO_WAVES][M5_STAGE];
    int32_t v2[MO_WAVES][M5_Q];
    int32_t u[MO_WAVES][M5_Q];
    int32_t m[MO_WAVES][M5_Q];   // pair mask of the 4-set | p(3) << 8
    uint32_t n[MO_WAVES];
    unsigned long long cnt[21];
};

__device__ __forceinline__ bool adj_g(const MotifArgs& A, int32_t a, int32_t u) {
    const int64_t r0 = A.rp[a];
    return member(A.col + r0, (int32_t)(A.rp[a + 1] - r0), u);
}

// the lists of v0 and v1 (shared by the wave's entries): LDS copies or the CSR
struct M5Lists {
    const int32_t* l0;
    const int32_t* l1;
    int32_t d0, d1;
};

// canonical extensions w of the 4-set (v0, v1, x2, x3) with pair mask m4 and
// p(3) = p3, from the lists of positions p3..3
__device__ __forceinline__ void last5_walk(const MotifArgs& A, const M5Lists& S, const int8_t* __restrict__ lut,
                                           int32_t v0, int32_t v1, int32_t x2, int32_t x3, int m4, int p3,
                                           unsigned long long* cnt, uint64_t& walked) {
    for (int J = p3; J < 4; ++J) {
        const int32_t xj = J == 0 ? v0 : (J == 1 ? v1 : (J == 2 ? x2 : x3));
        const int64_t t0 = A.rp[xj], t1 = A.rp[xj + 1];
        walked += (uint64_t)(t1 - t0);
        for (int64_t t = t0; t < t1; ++t) {
            const int32_t w = A.col[t];
            if (w <= v0 || w == v1 || w == x2 || w == x3) continue;
            if (J == p3 && w <= x3) continue;
            if (J > 0 && member(S.l0, S.d0, w)) continue;
            if (J > 1 && member(S.l1, S.d1, w)) continue;
            if (J > 2 && adj_g(A, x2, w)) continue;
            const int a0 = J == 0 ? 1 : 0;
            const int a1 = J == 1 ? 1 : (J < 1 ? (int)member(S.l1, S.d1, w) : 0);
            const int a2 = J == 2 ? 1 : (J < 2 ? (int)adj_g(A, x2, w) : 0);
            const int a3 = J == 3 ? 1 : (int)adj_g(A, x3, w);
            const int c = lut[m4 | (a0 << 6) | (a1 << 7) | (a2 << 8) | (a3 << 9)];
            if (c >= 0) atomicAdd(&cnt[c], 1ull);   // always connected; the test keeps LDS in bounds
        }
    }
}

__global__ __launch_bounds__(MO_THREADS) void k_motif_last5(MotifArgs A, const int8_t* __restrict__ lut) {
    __shared__ M5Lds L;
    const int w = threadIdx.x / WAVE;
    for (int i = threadIdx.x; i < 21; i += blockDim.x) L.cnt[i] = 0;
    __syncthreads();
    uint64_t walked = 0, n2 = 0, n3 = 0;   // work record: list elements walked, entries
    QueueCursor cur = queue_start();
    int64_t it_end = 0;
    for (int64_t it = queue_next(A.Q, cur, it_end); it >= 0; it = queue_next(A.Q, cur, it_end)) {
        for (int64_t j = it; j < it_end; ++j) {
            const uint64_t item = A.items[j];
            const int64_t p = item_seg(item);
            const int32_t x = (int32_t)item_round(item) * WAVE + lane();
            const int32_t s = (int32_t)(A.seg2[p + 1] - A.seg2[p]);
            const int32_t v0 = A.l1_src[p], v1 = A.l1_dst[p];
            M5Lists S;
            {
                const int64_t r0 = A.rp[v0], q0 = A.rp[v1];
                S.d0 = (int32_t)(A.rp[v0 + 1] - r0);
                S.d1 = (int32_t)(A.rp[v1 + 1] - q0);
                S.l0 = A.col + r0;
                S.l1 = A.col + q0;
                if (S.d0 <= M5_STAGE) {
                    for (int i = lane(); i < S.d0; i += WAVE) L.s0[w][i] = A.col[r0 + i];
                    S.l0 = &L.s0[w][0];
                }
                if (S.d1 <= M5_STAGE) {
                    for (int i = lane(); i < S.d1; i += WAVE) L.s1[w][i] = A.col[q0 + i];
                    S.l1 = &L.s1[w][0];
                }
                __threadfence_block();
                wave_sync();
            }
            bool done = x >= s;
            int32_t v2 = 0;
            int m3 = 0, I = 3;
            int64_t t = 0, t1 = 0;
            if (!done) {
                const int64_t e = (int64_t)(A.seg2[p] - A.seg2_base) + x;
                v2 = A.vid2[e];
                const int code = A.code2[e];
                m3 = 1 | ((code & 1) << 1) | (((code >> 1) & 1) << 2);
                I = (code & 1) ? 0 : 1;   // p(2): v2's first adjacent position
                const int32_t vi = I == 0 ? v0 : v1;
                t = A.rp[vi];
                t1 = A.rp[vi + 1];
                walked += (uint64_t)(t1 - t);
                ++n2;
            }
            const int p2 = (I == 0) ? 0 : 1;
            while (ballot(!done) != 0ull) {
                if (lane() == 0) L.n[w] = 0u;
                __threadfence_block();
                wave_sync();
                // level 3: queue extensions u until the queue is full
                while (!done) {
                    if (t >= t1) {   // the next list: positions I + 1 .. 2
                        if (++I > 2) {
                            done = true;
                            break;
                        }
                        const int32_t vi = I == 1 ? v1 : v2;
                        t = A.rp[vi];
                        t1 = A.rp[vi + 1];
                        walked += (uint64_t)(t1 - t);
                        continue;
                    }
                    const int32_t u = A.col[t];
                    bool ok = u > v0 && u != v1 && u != v2 && !(I == p2 && u <= v2);
                    ok = ok && !(I > 0 && member(S.l0, S.d0, u)) && !(I > 1 && member(S.l1, S.d1, u));
                    if (ok) {
                        const int a0 = I == 0 ? 1 : 0;
                        const int a1 = I == 1 ? 1 : (I < 1 ? (int)member(S.l1, S.d1, u) : 0);
                        const int a2 = I == 2 ? 1 : (int)adj_g(A, v2, u);
                        const uint32_t slot = atomicAdd(&L.n[w], 1u);
                        if (slot >= (uint32_t)M5_Q) break;   // full: retry u next round
                        L.v2[w][slot] = v2;
                        L.u[w][slot] = u;
                        L.m[w][slot] = (m3 | (a0 << 3) | (a1 << 4) | (a2 << 5)) | (I << 8);
                        ++n3;
                    }
                    ++t;
                }
                __threadfence_block();
                wave_sync();
                // level 4: one queued 4-set per lane
                const uint32_t nq = min(L.n[w], (uint32_t)M5_Q);
                for (uint32_t q = lane(); q < nq; q += WAVE) {
                    const int mq = L.m[w][q];
                    last5_walk(A, S, lut, v0, v1, L.v2[w][q], L.u[w][q], mq & 255, mq >> 8, L.cnt, walked);
                }
                wave_sync();
            }
            wave_sync();   // the next item overwrites the staged lists
        }
    }
    const uint64_t ws = wave_sum_u64(walked), s2 = wave_sum_u64(n2), s3 = wave_sum_u64(n3);
    if (lane() == 0) {
        if (ws) atomicAdd(&A.out[24], (unsigned long long)ws);
        if (s2) atomicAdd(&A.out[25], (unsigned long long)s2);
        if (s3) atomicAdd(&A.out[26], (unsigned long long)s3);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 21; i += blockDim.x)
        if (L.cnt[i]) atomicAdd(&A.out[i], L.cnt[i]);
}

// The table of the classes of five vertices (see above), built once.
static const Motif5Table& motif5_table() {
    static const Motif5Table t = [] {
        Motif5Table r{};
        int pos[5] = {0, 1, 2, 3, 4};
        int best[1024];
        for (int m = 0; m < 1024; ++m) best[m] = 1024;
        do {   // every relabelling of the positions
            for (int m = 0; m < 1024; ++m) {
                int q = 0;
                for (int b = 1; b < 5; ++b)
                    for (int a = 0; a < b; ++a) {
                        if (!((m >> (b * (b - 1) / 2 + a)) & 1)) continue;
                        const int x = std::min(pos[a], pos[b]), y = std::max(pos[a], pos[b]);
                        q |= 1 << (y * (y - 1) / 2 + x);
                    }
                best[m] = std::min(best[m], q);
            }
        } while (std::next_permutation(pos, pos + 5));
        std::vector<int> classes;
        std::vector<bool> conn(1024);
        for (int m = 0; m < 1024; ++m) {
            int reach = 1;   // vertices reachable from position 0
            for (int round = 0; round < 4; ++round)
                for (int b = 1; b < 5; ++b)
                    for (int a = 0; a < b; ++a)
                        if (((m >> (b * (b - 1) / 2 + a)) & 1) && ((reach >> a) & 1 || (reach >> b) & 1))
                            reach |= (1 << a) | (1 << b);
            conn[m] = reach == 31;
            if (conn[m] && best[m] == m) classes.push_back(m);
        }
        std::sort(classes.begin(), classes.end(), [](int a, int b) {
            const int ea = __builtin_popcount(a), eb = __builtin_popcount(b);
            return ea != eb ? ea < eb : a < b;
        });
        for (int m = 0; m < 1024; ++m) {
            r.cls[m] = -1;
            if (!conn[m]) continue;
            const auto it = std::lower_bound(classes.begin(), classes.end(), best[m], [](int a, int b) {
                const int ea = __builtin_popcount(a), eb = __builtin_popcount(b);
                return ea != eb ? ea < eb : a < b;
            });
            r.cls[m] = (int8_t)(it - classes.begin());
        }
        for (size_t j = 0; j < classes.size(); ++j)   // subsets of each class's edges
            for (int m = classes[j]; m > 0; m = (m - 1) & classes[j])
                if (r.cls[m] >= 0) ++r.copies[r.cls[m]][j];
        return r;
    }();
    return t;
}

// ------------------------------------------------------------------ host

struct MotifRun {
    pg_graph* g;
    hipStream_t s;
    unsigned long long* out;    // 16 counters
    unsigned long long* qctr;
    int64_t waves;
    int blocks;
};

static MotifArgs base_args(const MotifView& V) {
    MotifArgs A{};
    A.rp = V.rp;
    A.col = V.col;
    A.l1_seg = V.ml1->seg.as<int64_t>();
    A.l1_src = V.ml1->src.as<int32_t>();
    A.l1_dst = V.ml1->dst.as<int32_t>();
    A.hub_id = V.ml1->hub_id.as<int32_t>();
    A.hub_bits = V.ml1->hub_bits.as<uint32_t>();
    A.hub_words = V.ml1->hub_words;
    return A;
}

__global__ __launch_bounds__(256) void k_hub_rows(int64_t n_hubs, const int32_t* __restrict__ hubs,
                                                  const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                  int64_t words, uint32_t* __restrict__ bits) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    for (int64_t h = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; h < n_hubs; h += waves) {
        const int32_t v = hubs[h];
        uint32_t* row = bits + h * words;
        for (int64_t j = rp[v] + lane(); j < rp[v + 1]; j += WAVE) {
            const uint32_t u = (uint32_t)col[j];
            atomicOr(row + (u >> 5), 1u << (u & 31));
        }
    }
}

// Dense adjacency rows for the vertices whose lists are too long to stage in
// LDS (degree > MO_STAGE), within a memory cap (the highest degrees first
// when the cap binds).
static void build_hubs(pg_graph* g, const MotifView& V) {
    MotifL1& L = *V.ml1;
    if (L.hubs_built) return;
    hipStream_t s = g->stream;
    const int64_t n = V.n;
    std::vector<int64_t> hrp((size_t)n + 1);
    PG_HIP(hipMemcpyAsync(hrp.data(), V.rp, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    const int64_t words = (n + 31) / 32;
    const uint64_t cap = std::min<uint64_t>(uint64_t(2) << 30, std::max<uint64_t>(g->budget / 8, 1));
    int64_t thr = MO_STAGE + 1;
    std::vector<int32_t> hubs;
    while (true) {
        hubs.clear();
        for (int64_t v = 0; v < n; ++v)
            if (hrp[v + 1] - hrp[v] >= thr) hubs.push_back((int32_t)v);
        if ((uint64_t)hubs.size() * (uint64_t)words * 4 <= cap) break;
        thr *= 2;
    }
    std::vector<int32_t> id((size_t)std::max<int64_t>(n, 1), -1);
    DevBuf hl;
    SettleOnError settle(s);
    for (size_t h = 0; h < hubs.size(); ++h) id[(size_t)hubs[h]] = (int32_t)h;
    L.hub_id.reserve(sizeof(int32_t) * id.size());
    PG_HIP(hipMemcpyAsync(L.hub_id.p, id.data(), sizeof(int32_t) * id.size(), hipMemcpyHostToDevice, s));
    L.n_hubs = (int64_t)hubs.size();
    L.hub_words = words;
    L.hub_bits.reserve(sizeof(uint32_t) * std::max<int64_t>(L.n_hubs * words, 1));
    if (L.n_hubs > 0) {
        hl.reserve(sizeof(int32_t) * hubs.size());
        PG_HIP(hipMemcpyAsync(hl.p, hubs.data(), sizeof(int32_t) * hubs.size(), hipMemcpyHostToDevice, s));
        fill_u32(L.hub_bits.as<uint32_t>(), L.n_hubs * words, 0, s);
        k_hub_rows<<<(unsigned)std::min<int64_t>((L.n_hubs + 3) / 4, 4096), 256, 0, s>>>(
            L.n_hubs, hl.as<int32_t>(), V.rp, V.col, words, L.hub_bits.as<uint32_t>());
        PG_HIP(hipGetLastError());
        PG_HIP(hipStreamSynchronize(s));
    }
    PG_HIP(hipStreamSynchronize(s));
    L.hubs_built = true;
}

static void set_queue(MotifRun& R, MotifArgs& A, const uint64_t* items, int64_t n_items) {
    fill_u64(reinterpret_cast<uint64_t*>(R.qctr), Q_WORDS, 0, R.s);
    A.Q.next = R.qctr;
    A.Q.n_items = n_items;
    A.Q.chunk = n_items >= R.waves * 64 ? 4 : 1;
    A.items = items;
    A.out = R.out;
}

// a level-1 pass over the vertices [v_lo, v_hi), in items of 64 L1 entries
template <int MODE>
static void launch_l1(MotifRun& R, MotifArgs A, int64_t v_lo, int64_t v_hi, const char* name, double units) {
    if (v_hi <= v_lo) return;
    Arena& ar = R.g->arena;
    const size_t mk = ar.mark();
    uint64_t* items = nullptr;
    const int64_t m = round_items(A.l1_seg, v_lo, v_hi - v_lo, WAVE, ar, R.s, &items);
    if (m > 0) {
        set_queue(R, A, items, m);
        ProfScope ps(name, R.s, units);
        k_motif_l1<MODE><<<R.blocks, MO_THREADS, 0, R.s>>>(A);
        PG_HIP(hipGetLastError());
    }
    ar.reset(mk);
}

// first vertex whose L1 segment holds entry x: largest v with l1_seg[v] <= x
__global__ void k_vertex_of_entry(const int64_t* __restrict__ seg, int64_t n, const int64_t* __restrict__ xs,
                                  int64_t nq, int64_t* __restrict__ out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nq) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (seg[mid] <= xs[i]) lo = mid; else hi = mid - 1;
    }
    out[i] = lo;
}

__global__ void k_chunk_entries(const uint64_t* __restrict__ start, int64_t m, uint64_t cap, int64_t nb,
                                int64_t* __restrict__ out_c, uint64_t* __restrict__ out_s) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j > nb) return;
    int64_t c;
    if (j == 0) c = 0;
    else if (j == nb) c = m;
    else {
        const uint64_t target = (uint64_t)j * cap;
        int64_t lo = 0, hi = m;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (start[mid] <= target) lo = mid; else hi = mid - 1;
        }
        c = lo;
    }
    out_c[j] = c;
    out_s[j] = start[c];
}

static void count_motifs5(pg_graph* g, uint64_t* counts) {
    if (count_motifs5_sums(g, motif5_table(), counts)) return;
    const MotifView V = motif_view(g, false);
    build_motif_l1(g, V);
    build_hubs(g, V);
    const int64_t E = V.ml1->n_edges;
    for (int i = 0; i < 21; ++i) counts[i] = 0;
    if (E == 0) return;
    hipStream_t s = g->stream;
    Arena& ar = g->arena;
    MotifRun R;
    R.g = g;
    R.s = s;
    R.waves = grid_waves(16);
    R.blocks = (int)(R.waves / MO_WAVES);
    uint64_t* small = push<uint64_t>(ar, 32 + Q_WORDS);
    R.out = reinterpret_cast<unsigned long long*>(small);
    R.qctr = reinterpret_cast<unsigned long long*>(small + 32);
    fill_u64(small, 32, 0, s);
    // lanes wait on dependent searches, so more waves per CU hide them: as many
    // workgroups per CU as its LDS and registers let reside, up to
    // MO5_WAVES_PER_CU waves
    int blocks5 = (int)(grid_waves(MO5_WAVES_PER_CU) / MO_WAVES);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_motif_last5, MO_THREADS, 0) == hipSuccess && per_cu > 0)
        blocks5 = device_info().n_cu * std::min(per_cu, MO5_WAVES_PER_CU / MO_WAVES);
    else
        (void)hipGetLastError();
    int8_t* lut5 = push<int8_t>(ar, 1024);
    PG_HIP(hipMemcpyAsync(lut5, motif5_table().cls, 1024, hipMemcpyHostToDevice, s));
    MotifArgs A = base_args(V);
    A.x_lo = 0;
    A.x_hi = E;
    // level 2: count pass -> scan -> write, in chunks of L1 entries that fit the budget
    uint32_t* cnt = push<uint32_t>(ar, E);
    uint64_t* start = push<uint64_t>(ar, E + 1);
    A.count = cnt;
    launch_l1<ML1_COUNT>(R, A, 0, g->n, "motif_count", (double)E);
    scan_u32(cnt, E, start, ar, s);
    const uint64_t total = read_u64(start + E, s);
    const uint64_t per = 5;   // vid + code per L2 entry
    const uint64_t room = g->budget > ar.mark() ? g->budget - ar.mark() : 0;
    const uint64_t cap = std::max<uint64_t>(room / per, (uint64_t)(2 * g->max_deg + 1));
    const int64_t nb = total == 0 ? 0 : (int64_t)((total + cap - 1) / cap);
    std::vector<int64_t> hc(nb + 1, 0), hv(nb + 1, 0);
    std::vector<uint64_t> hs(nb + 1, 0);
    if (nb >= 1) {
        const size_t mk = ar.mark();
        int64_t* dc = push<int64_t>(ar, nb + 1);
        uint64_t* ds = push<uint64_t>(ar, nb + 1);
        int64_t* dv = push<int64_t>(ar, nb + 1);
        k_chunk_entries<<<(unsigned)((nb + 256) / 256), 256, 0, s>>>(start, E, cap, nb, dc, ds);
        PG_HIP(hipGetLastError());
        k_vertex_of_entry<<<(unsigned)((nb + 256) / 256), 256, 0, s>>>(A.l1_seg, g->n, dc, nb + 1, dv);
        PG_HIP(hipGetLastError());
        PG_HIP(hipMemcpyAsync(hc.data(), dc, sizeof(int64_t) * (nb + 1), hipMemcpyDeviceToHost, s));
        PG_HIP(hipMemcpyAsync(hs.data(), ds, sizeof(uint64_t) * (nb + 1), hipMemcpyDeviceToHost, s));
        PG_HIP(hipMemcpyAsync(hv.data(), dv, sizeof(int64_t) * (nb + 1), hipMemcpyDeviceToHost, s));
        PG_HIP(hipStreamSynchronize(s));
        ar.reset(mk);
    }
    uint64_t biggest = 0;
    for (int64_t j = 0; j < nb; ++j) biggest = std::max<uint64_t>(biggest, hs[j + 1] - hs[j]);
    int32_t* vid2 = push<int32_t>(ar, std::max<uint64_t>(biggest, 1));
    uint8_t* code2 = push<uint8_t>(ar, std::max<uint64_t>(biggest, 1));
    for (int64_t j = 0; j < nb; ++j) {
        const int64_t c0 = hc[j], c1 = hc[j + 1];
        if (c1 <= c0) continue;
        MotifArgs W = A;
        W.x_lo = c0;
        W.x_hi = c1;
        W.start = start;
        W.start_base = hs[j];
        W.out_vid = vid2;
        W.out_code = code2;
        const int64_t v_lo = hv[j];
        const int64_t v_hi = (j + 1 == nb) ? g->n : std::min<int64_t>(g->n, hv[j + 1] + 1);
        launch_l1<ML1_WRITE>(R, W, v_lo, v_hi, "motif_write", (double)(hs[j + 1] - hs[j]));
        // fused last level over the L1 entries [c0, c1) (segments of L2)
        MotifArgs L = A;
        L.seg2 = start;
        L.seg2_base = hs[j];
        L.vid2 = vid2;
        L.code2 = code2;
        const size_t mk = ar.mark();
        uint64_t* items = nullptr;
        const int64_t m = round_items(start, c0, c1 - c0, WAVE, ar, s, &items);
        if (m > 0) {
            set_queue(R, L, items, m);
            ProfScope ps("motif_last", s, 0.0);
            k_motif_last5<<<blocks5, MO_THREADS, 0, s>>>(L, lut5);
            PG_HIP(hipGetLastError());
        }
        ar.reset(mk);
    }
    uint64_t h[32];
    PG_HIP(hipMemcpyAsync(h, small, sizeof(h), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    for (int i = 0; i < 21; ++i) counts[i] = h[i];
    if (prof_on()) {
        // per level-2 entry its SoA entry and a row-pointer pair
        // (16 B), per level-3 extension a row-pointer pair (16 B), and 4 B
        // per element of every list walked at levels 3 and 4
        ProfScope ps("motif_last_work", s, 16.0 * (double)(h[25] + h[26]) + 4.0 * (double)h[24]);
    }
}

void count_motifs(pg_graph* g, int k, uint64_t* counts) {
    PG_REQUIRE(k >= 3 && k <= 5, PG_EUNSUPPORTED, "motif size must be 3, 4 or 5");
    if (k == 3) count_motifs3(g, counts);
    else if (k == 4) count_motifs4(g, counts);
    else count_motifs5(g, counts);
}

}  // namespace pg
