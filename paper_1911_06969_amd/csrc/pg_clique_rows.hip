// The count pass of the clique kernels by tables: rows (or triangles) of roots
// whose out-lists lie close enough together.
//
// Entry i of a root r streams out(S[i]), S = out(r), and asks for each element
// whether it is in S, and where.  Ranks are dense, so a list of D vertices among
// the W thousand ranks up to its last one fits a bitmap of its range: word
// (u - S[0]) / 32 holds 32 ranks' bits and the number of S's elements below them,
// and one 8-byte read of LDS answers both questions.  A search of S takes log2(D)
// dependent reads instead, each with an add, a compare and a select.
//
// A workgroup lays out the table of an item's root, takes the item's entries one
// by one, a wave each, and clears the words it set.
//
// Measured on R-MAT scale 21, edge factor 13 (7.1 billion elements streamed, 6.4
// of them at roots that take tables): 8.25 ms for the pass by searches, 6.6 ms
// now (small tables 4.25, large 1.19, searches for what is left 1.18).  Bound by
// instruction issue: about 17 vector and 23 scalar instructions per 64 elements.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pg_clique.h"
#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

// Looks up NK rows of 64 elements; hits set bits of the LDS row (ROWS).
// Returns the number of hits (wave-uniform).
template <bool ROWS, int NK>
__device__ __forceinline__ uint32_t table_keys(const uint2* tab, uint32_t words, uint32_t base,
                                               const int32_t (&u)[BM_UNROLL], uint32_t* row) {
    uint32_t d[NK];
    uint2 t[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) {
        d[q] = (uint32_t)u[q] - base;
        t[q] = tab[min(d[q] >> 5, words)];   // the word past the table is empty
    }
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < NK; ++q) {
        const bool f = (t[q].x >> (d[q] & 31)) & 1u;
        c += (uint32_t)popc64(ballot(f));
        if (ROWS && f) {
            const uint32_t pos = t[q].y + (uint32_t)__popc(t[q].x & ((1u << (d[q] & 31)) - 1u));
            atomicOr(&row[pos >> 5], 1u << (pos & 31));
        }
    }
    return c;
}

template <bool ROWS, int CLS>
__global__ __launch_bounds__(CLS == 0 ? 256 : 512, CLS == 0 ? 7 : 6) void k_rows_table(XcdQueue Q,
                                                                                      const uint64_t* __restrict__ items,
                                                                                      CountArgs A) {
    constexpr int THREADS = CLS == 0 ? 256 : 512;
    constexpr int WORDS = CR_WORDS[CLS];
    constexpr int PER = (BM_MAXD + THREADS - 1) / THREADS;   // list elements per thread
    __shared__ uint2 tab[WORDS + 1];
    __shared__ uint32_t rows[THREADS / WAVE][2 * BM_W];
    __shared__ int64_t s_b, s_base;
    __shared__ int32_t s_d, s_x0, s_entry;
    const int w = threadIdx.x / WAVE;
    uint32_t* row = rows[w];
    for (int k = threadIdx.x; k <= WORDS; k += THREADS) tab[k] = make_uint2(0u, 0u);
    if (lane() < 2 * BM_W) row[lane()] = 0u;   // every entry leaves it zero again
    uint64_t streamed = 0, found = 0;          // wave-uniform
    QueueCursor cur = queue_start(1);
    // the next item, by wave 0: s_d = 0 after the last
    auto fetch = [&]() {
        int64_t end = 0;
        const int64_t it = queue_next(Q, cur, end);
        if (lane() == 0) {
            s_d = 0;
            if (it >= 0) {
                const uint64_t item = items[Q.n_items - 1 - it];
                const int64_t r = item_seg(item);
                s_b = A.rp[r];
                s_d = (int32_t)(A.rp[r + 1] - A.rp[r]);
                s_x0 = (int32_t)item_round(item) * A.round;
                if (ROWS) s_base = (int64_t)A.moff[r];
            }
        }
    };
    if (w == 0) fetch();
    while (true) {
        __syncthreads();   // the item is known, the table empty
        const int64_t b = uniform64(s_b);
        const int32_t d = uniform(s_d), x0 = uniform(s_x0);
        const int64_t mbase = ROWS ? uniform64(s_base) : 0;
        if (d == 0) break;
        const int nx = min(A.round, d - x0);
        const int32_t* S = A.col + b;
        const int32_t s_last = uniform(S[d - 1]);
        const uint32_t base = (uint32_t)uniform(S[0]) & ~31u;
        // out-list bounds of the item's entries, one per lane, in every wave
        const int32_t xl = x0 + lane();
        int64_t lo = 0;
        int32_t nl = 0;
        if (lane() < nx && xl < d - 1) {
            const int32_t v = S[xl];
            lo = A.rp[v];
            nl = (int32_t)(A.rp[v + 1] - lo);
        }
        uint32_t at[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = (int)threadIdx.x + q * THREADS;
            at[q] = WORDS;
            if (k < d) {
                const uint32_t u = (uint32_t)S[k] - base;
                at[q] = u >> 5;
                atomicOr(&tab[at[q]].x, 1u << (u & 31));
                // the first element of a word counts those before it
                if (k == 0 || ((uint32_t)S[k - 1] - base) >> 5 != at[q]) tab[at[q]].y = (uint32_t)k;
            }
        }
        if (threadIdx.x == 0) s_entry = 0;
        __syncthreads();   // the table is complete, the item read
        if (w == 0) fetch();
        const int W = (d + 63) >> 6;
        auto look = [&](const int32_t (&u)[BM_UNROLL], int n) -> uint32_t {
            if (n == 4) return table_keys<ROWS, 4>(tab, WORDS, base, u, row);
            if (n == 3) return table_keys<ROWS, 3>(tab, WORDS, base, u, row);
            if (n == 2) return table_keys<ROWS, 2>(tab, WORDS, base, u, row);
            return table_keys<ROWS, 1>(tab, WORDS, base, u, row);
        };
        while (true) {
            int xi = 0;
            if (lane() == 0) xi = atomicAdd(&s_entry, 1);
            xi = uniform(xi);
            if (xi >= nx) break;
            const int64_t l = (int64_t)readlane64((uint64_t)lo, xi);
            const int64_t n_cand = readlane(nl, xi);
            uint32_t c = 0;
            if (n_cand > 0) c = stream_list(A.col + l, n_cand, s_last, streamed, look);
            if constexpr (!ROWS) found += c;
            else {
                wave_sync();   // every lane's hits are in the row
                if (lane() < W) {
                    A.M[mbase + (int64_t)(x0 + xi) * W + lane()] =
                        (uint64_t)row[2 * lane()] | ((uint64_t)row[2 * lane() + 1] << 32);
                    row[2 * lane()] = 0u;
                    row[2 * lane() + 1] = 0u;
                }
                if (A.count && lane() == 0) {
                    A.count[b + x0 + xi] = c;
                    A.info[b + x0 + xi] = row_info((uint64_t)mbase, x0 + xi, W);
                }
                wave_sync();   // cleared before the next entry's hits
            }
        }
        __syncthreads();   // the table is read
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (at[q] < WORDS) tab[at[q]] = make_uint2(0u, 0u);
    }
    if (lane() == 0) add_stat(A.stats, 3, streamed);
    if (!ROWS && lane() == 0) add_stat(A.stats, 0, found);
}

void count_rows_table(pg_graph* g, int c, const CountArgs& A, unsigned long long* queue) {
    const MaskPlan& P = g->dag.plan;
    if (P.items[c] == 0) return;
    hipStream_t s = g->stream;
    XcdQueue Q;
    Q.next = queue;
    Q.n_items = P.items[c];
    const uint64_t* items = P.item[c].as<uint64_t>();
    const int threads = c == 0 ? 256 : 512;
    const auto kernel = c == 0 ? (A.M ? k_rows_table<true, 0> : k_rows_table<false, 0>)
                               : (A.M ? k_rows_table<true, 1> : k_rows_table<false, 1>);
    const unsigned blocks = queue_blocks(kernel, threads, 0, P.items[c]);
    Q.chunk = queue_chunk(Q.n_items, blocks, 1);
    kernel<<<blocks, threads, 0, s>>>(Q, items, A);
    PG_HIP(hipGetLastError());
}

}  // namespace pg
