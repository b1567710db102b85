// The count pass of the clique kernels: rows (or triangles) by the middle vertex.
//
// Row x of a root r asks which of the later vertices of out(r) are out-neighbours of
// v = out(r)[x].  A work item holds out(v) and takes the entries (r, x) of the DAG's
// in-list of v: for each, 64 later vertices of out(r) at a time, a lane each, and the
// ballot of the answers is the row's word.  So an entry reads the rest of its root's
// list, |out(r)| - x - 1 elements; taking the entries by root instead reads out(v) up to
// the root's last vertex, 7.1 billion elements against 2.0 on R-MAT scale 21, edge
// factor 13, and has to find the places of those that are in out(r).
//
// out(v) lies in LDS as a bitmap over its ids (ranks are dense), or, where these are
// too far apart or the entries too few to pay for it, in a register, an id per lane.
// Longer lists of ids too far apart lie in LDS as a bitmap over two hashes of the ids, and
// an element whose bits are both set (one in 200,000 of those that are not in a list of
// 75) is looked up in the list.  A million vertices of 150 random neighbours, triangles:
// 7.2 ms a call (one hash 8.4; lists of up to 64 compared in registers and longer ones
// searched 21.6; by root 12.7).
//
// Measured on that graph, with 25 million entries and 52 million words: 3.4 ms (bitmaps
// 2.93, registers 0.44); by root, 8.25 ms with searches of out(r), 6.6 with bitmaps of
// it.  Bound by the lists that come from beyond the L2s, 16 GB or 5.4 TB/s (21 GB with
// the items in the order of v), and by issue, 60 % of the time.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pg_clique.h"
#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

namespace {

constexpr int RT_THREADS = 256;
constexpr int RT_WAVES = RT_THREADS / WAVE;
constexpr int RT_PER = RT_WAVES * WAVE;   // entries of a table item
constexpr int RT_MIN_IN = 8;              // fewest entries that a bitmap is laid out for
constexpr int RT_WORDS = 2560;            // of 32 ids: 10 KB, 82 thousand ids
// Lists too far apart for a bitmap are hashed from this length on for so many entries,
// past 64 in any case.  Random graphs of a million vertices of 40, 70, 100 neighbours,
// us, with (8, 32) 1,834, 3,425, 5,254; (16, 32) 1,727, 3,449, 5,512; (16, 16) 1,887,
// 3,122, 5,160; (32, 64) 1,724, -, 9,147.
constexpr int RT_HASH_MIN_D = 16;
constexpr int RT_HASH_MIN_IN = 32;
constexpr int RT_HASH_WORDS = 2048;       // 65,536 hashes: 8 KB
enum { RC_TABLE = 0, RC_LIST, RC_HASH };  // how an item's list is held
__device__ __forceinline__ uint32_t rt_hash(uint32_t u) { return (u * 0x9E3779B1u) >> 16; }
__device__ __forceinline__ uint32_t rt_hash2(uint32_t u) { return (u * 0x85EBCA6Bu) >> 16; }
constexpr int RT_DEEP = 8;                // row words of a step: by bitmap
constexpr int RT_FEW = 4;                 // ... by list: most items have that many or fewer

// the entries of a wave, one per lane
struct Entries {
    int32_t e;          // DAG edge (r, v)
    int32_t at;         // first element of the row's first word, in col
    int32_t left;       // elements from there to the end of out(r)
    int32_t words;      // row words from there (0: no entry)
    int64_t out;        // the first word's place in M
    int64_t base;       // of r's block in M
    int32_t x, W;
};

template <bool ROWS>
__device__ __forceinline__ Entries load_entry(const CountArgs& A, int64_t k, bool on) {
    Entries E{0, 0, 0, 0, 0, 0, 0, 0};
    if (on) {
        E.e = A.in_edge[k];
        const int32_t r = A.in_src[k];
        const int64_t b = A.rp[r];
        const int32_t d = (int32_t)(A.rp[r + 1] - b);
        E.x = E.e - (int32_t)b;
        if (E.x + 1 >= d || d > BM_MAXD) return E;   // no row to fill
        E.W = (d + 63) >> 6;
        const int32_t q = (E.x + 1) >> 6;   // words below hold places up to x: empty
        E.at = (int32_t)b + 64 * q;
        E.left = d - 64 * q;
        E.words = E.W - q;
        if (ROWS) {
            E.base = (int64_t)A.moff[r];
            E.out = E.base + (int64_t)E.x * E.W + q;
        }
    }
    return E;
}

// Rows of a wave's entries.  find(u, f): which of DEEP elements per lane are in out(v); places up to x hold ids up to v, which are not.
template <bool ROWS, int DEEP, class Find>
__device__ __forceinline__ uint64_t entry_rows(const CountArgs& A, const Entries& E, Find find) {
    uint64_t found = 0;    // wave-uniform
    uint32_t mine = 0;     // hits of the lane's entry
    for (int j = 0;; ++j) {
        uint64_t todo = ballot(E.words > j);
        if (!todo) break;
        const int32_t at = E.at + 64 * j, left = E.left - 64 * j;
        uint32_t lo = 0, hi = 0;   // word j of the lane's row
        while (todo) {
            int l[DEEP];
            uint32_t u[DEEP];
            bool f[DEEP];
            const int m = min(DEEP, popc64(todo));
            // all loads of the step first (past the list's end: masked below;
            // col has 64 elements more)
#pragma unroll
            for (int i = 0; i < DEEP; ++i) {
                l[i] = 0;
                u[i] = 0;
                if (i < m) {
                    l[i] = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    u[i] = (uint32_t)A.col[(int64_t)readlane(at, l[i]) + lane()];
                }
            }
            find(u, f);
#pragma unroll
            for (int i = 0; i < DEEP; ++i) {
                if (i < m) {
                    const int32_t rest = readlane(left, l[i]);
                    uint64_t b = ballot(f[i]);
                    if (rest < WAVE) b &= (1ull << rest) - 1ull;
                    if constexpr (ROWS) {
                        if (lane() == l[i]) {
                            lo = (uint32_t)b;
                            hi = (uint32_t)(b >> 32);
                        }
                    } else {
                        found += (uint64_t)popc64(b);
                    }
                }
            }
        }
        if (ROWS && (lo | hi)) {   // the rows are zero before
            A.M[E.out + j] = (uint64_t)lo | ((uint64_t)hi << 32);
            mine += (uint32_t)(__popc(lo) + __popc(hi));
        }
    }
    if (ROWS && A.count && E.words > 0) {
        A.count[E.e] = mine;
        if (A.info) A.info[E.e] = row_info((uint64_t)E.base, E.x, E.W);
    }
    return found;
}

}  // namespace

// A workgroup lays out the bitmap of an item's vertex (item: v and the round of
// RT_PER entries of its in-list), its waves take a quarter of the entries each, and
// the words it set are cleared.  Wave 0 fetches the next item meanwhile.
template <bool ROWS, bool HASH>
__global__ __launch_bounds__(RT_THREADS, 8) void k_rows_table(XcdQueue Q, const uint64_t* __restrict__ items,
                                                              CountArgs A) {
    constexpr int WORDS = HASH ? RT_HASH_WORDS : RT_WORDS + 1;
    __shared__ uint32_t tab[WORDS];
    __shared__ int64_t s_lo, s_k;
    __shared__ int32_t s_d, s_n;
    const int w = threadIdx.x / WAVE;
    for (int k = threadIdx.x; k < WORDS; k += RT_THREADS) tab[k] = 0u;
    uint64_t found = 0, read = 0;
    QueueCursor cur = queue_start(1);
    // the next item, by wave 0: s_d = 0 after the last
    auto fetch = [&]() {
        int64_t end = 0;
        const int64_t it = queue_next(Q, cur, end);
        if (lane() == 0) {
            s_d = 0;
            if (it >= 0) {
                const uint64_t item = items[Q.n_items - 1 - it];
                const int64_t v = item_seg(item);
                s_lo = A.rp[v];
                s_d = (int32_t)(A.rp[v + 1] - A.rp[v]);
                s_k = A.in_rp[v] + item_round(item) * RT_PER;
                s_n = (int32_t)min64(RT_PER, A.in_rp[v + 1] - s_k);
            }
        }
    };
    if (w == 0) fetch();
    while (true) {
        __syncthreads();   // the item is known, the bitmap empty
        const int32_t* S = A.col + uniform64(s_lo);
        const int64_t k0 = uniform64(s_k);
        const int32_t d = uniform(s_d), n = uniform(s_n);
        if (d == 0) break;
        const int32_t per = (n + RT_WAVES - 1) / RT_WAVES, mine = w * per + lane();
        const Entries E = load_entry<ROWS>(A, k0 + mine, lane() < per && mine < n);
        const uint32_t base = HASH ? 0u : (uint32_t)uniform(S[0]) & ~31u;
        for (int k = threadIdx.x; k < d; k += RT_THREADS) {
            if constexpr (HASH) {
                const uint32_t h = rt_hash((uint32_t)S[k]), h2 = rt_hash2((uint32_t)S[k]);
                atomicOr(&tab[h >> 5], 1u << (h & 31));
                atomicOr(&tab[h2 >> 5], 1u << (h2 & 31));
            } else {
                const uint32_t u = (uint32_t)S[k] - base;
                atomicOr(&tab[u >> 5], 1u << (u & 31));
            }
        }
        __syncthreads();   // the bitmap is complete, the item read
        if (w == 0) fetch();
        read += (uint64_t)max(E.left, 0);
        found += entry_rows<ROWS, RT_DEEP>(A, E, [&](const uint32_t (&u)[RT_DEEP], bool (&f)[RT_DEEP]) {
            uint32_t t[RT_DEEP];
            if constexpr (HASH) {
#pragma unroll
                for (int i = 0; i < RT_DEEP; ++i) t[i] = tab[rt_hash(u[i]) >> 5];
#pragma unroll
                for (int i = 0; i < RT_DEEP; ++i) f[i] = (t[i] >> (rt_hash(u[i]) & 31)) & 1u;
#pragma unroll
                for (int i = 0; i < RT_DEEP; ++i)
                    if (ballot(f[i]) != 0ull) {
                        const uint32_t h = rt_hash2(u[i]);
                        f[i] = f[i] && ((tab[h >> 5] >> (h & 31)) & 1u);
                        if (ballot(f[i]) != 0ull) f[i] = f[i] && contains(S, d, (int32_t)u[i]);
                    }
            } else {
#pragma unroll
                for (int i = 0; i < RT_DEEP; ++i) t[i] = tab[min((u[i] - base) >> 5, (uint32_t)RT_WORDS)];
#pragma unroll
                for (int i = 0; i < RT_DEEP; ++i) f[i] = (t[i] >> (u[i] & 31)) & 1u;   // base is a multiple of 32
            }
        });
        __syncthreads();   // the bitmap is read
        for (int k = threadIdx.x; k < d; k += RT_THREADS) {
            if constexpr (HASH) {
                tab[rt_hash((uint32_t)S[k]) >> 5] = 0u;
                tab[rt_hash2((uint32_t)S[k]) >> 5] = 0u;
            } else {
                tab[((uint32_t)S[k] - base) >> 5] = 0u;
            }
        }
    }
    read = wave_sum_u64(read);
    if (lane() == 0) {
        add_stat(A.stats, 3, read);
        if (!ROWS) add_stat(A.stats, 0, found);
    }
}

// A wave per item (v and a round of 64 entries).
template <bool ROWS>
__global__ __launch_bounds__(RT_THREADS, 8) void k_rows_list(XcdQueue Q, const uint64_t* __restrict__ items,
                                                             CountArgs A) {
    uint64_t found = 0, read = 0;
    QueueCursor cur = queue_start();
    int64_t end = 0;
    for (int64_t it = queue_next(Q, cur, end); it >= 0; it = queue_next(Q, cur, end))
        for (; it < end; ++it) {
            const uint64_t item = items[it];
            const int64_t v = uniform64(item_seg(item));
            const int64_t s0 = uniform64(A.rp[v]);
            const int32_t d = uniform((int32_t)(A.rp[v + 1] - s0));
            const int64_t k = A.in_rp[v] + item_round(item) * WAVE + lane();
            const Entries E = load_entry<ROWS>(A, k, k < A.in_rp[v + 1]);
            read += (uint64_t)max(E.left, 0);
            const uint32_t own = lane() < d ? (uint32_t)A.col[s0 + lane()] : 0u;   // ids in lists are 1 or more
            found += entry_rows<ROWS, RT_FEW>(A, E, [&](const uint32_t (&u)[RT_FEW], bool (&f)[RT_FEW]) {
                if (d <= WAVE) {
                    uint32_t miss[RT_FEW];   // 0 once an id equals the element
#pragma unroll
                    for (int i = 0; i < RT_FEW; ++i) miss[i] = ~0u;
                    for (int j = 0; j < d; ++j) {
                        const uint32_t x = (uint32_t)readlane((int32_t)own, j);
#pragma unroll
                        for (int i = 0; i < RT_FEW; ++i) miss[i] = min(miss[i], u[i] ^ x);
                    }
#pragma unroll
                    for (int i = 0; i < RT_FEW; ++i) f[i] = miss[i] == 0u;
                } else {
#pragma unroll
                    for (int i = 0; i < RT_FEW; ++i) f[i] = contains(A.col + s0, d, (int32_t)u[i]);
                }
            });
        }
    read = wave_sum_u64(read);
    if (lane() == 0) {
        add_stat(A.stats, 3, read);
        if (!ROWS) add_stat(A.stats, 0, found);
    }
}

// In-list keys (large graphs): (v << 32 | e) of every edge e = (r, v) with a row to fill: r light
// and with out-neighbours after v, v with any.  The others sort last (v = n).
__global__ void k_in_keys(int64_t n, int64_t m, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                          const int32_t* __restrict__ src, uint64_t* __restrict__ keys) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = src[e], v = col[e];
        const int64_t b = rp[r], end = rp[r + 1];
        const bool on = end - b <= BM_MAXD && e + 1 < end && rp[v + 1] > rp[v];
        keys[e] = ((on ? (uint64_t)(uint32_t)v : (uint64_t)n) << 32) | (uint64_t)e;
    }
}

__global__ void k_in_rows(int64_t n, int64_t m, const uint64_t* __restrict__ keys, int64_t* __restrict__ in_rp) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v <= n; v += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = m;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((keys[mid] >> 32) < (uint64_t)v) lo = mid + 1; else hi = mid;
        }
        in_rp[v] = lo;
    }
}

__global__ void k_in_lists(int64_t m, const uint64_t* __restrict__ keys, const int32_t* __restrict__ src,
                           int32_t* __restrict__ in_edge, int32_t* __restrict__ in_src) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < m; k += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t e = (uint32_t)keys[k];
        in_edge[k] = (int32_t)e;
        in_src[k] = src[e];
    }
}

// Entries of v by how its list is held.  A bitmap from RT_MIN_IN entries on: it costs a
// workgroup two turns of its barriers, about as much as 64 words' looks at a list in
// registers; a hashed one for longer lists.  table, list, hash: v's items of each kind.
__global__ void k_in_class(int64_t n, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                           const int64_t* __restrict__ in_rp, uint32_t* __restrict__ table, uint32_t* __restrict__ list,
                           uint32_t* __restrict__ hash) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t c = rp[v + 1] > rp[v] ? (uint32_t)(in_rp[v + 1] - in_rp[v]) : 0u;
        int how = RC_LIST;
        if (c >= RT_MIN_IN) {
            if ((col[rp[v + 1] - 1] >> 5) - (col[rp[v]] >> 5) < RT_WORDS) how = RC_TABLE;
            else if (rp[v + 1] - rp[v] > (c >= RT_HASH_MIN_IN ? RT_HASH_MIN_D : WAVE)) how = RC_HASH;
        }
        const uint32_t wide = (c + RT_PER - 1) / RT_PER;
        table[v] = how == RC_TABLE ? wide : 0u;
        list[v] = how == RC_LIST ? (c + WAVE - 1) / WAVE : 0u;
        hash[v] = how == RC_HASH ? wide : 0u;
    }
}

__global__ void k_in_items(int64_t n, const uint64_t* __restrict__ pos, uint64_t* __restrict__ items) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        for (uint64_t i = pos[v]; i < pos[v + 1]; ++i) items[i] = ((uint64_t)v << ROUND_BITS) | (i - pos[v]);
}

// (root of the item's first entry << 32 | item)
__global__ void k_item_keys(int64_t n_items, const uint64_t* __restrict__ items, const int64_t* __restrict__ in_rp,
                            const int32_t* __restrict__ in_src, uint64_t* __restrict__ keys) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_items; i += (int64_t)gridDim.x * blockDim.x)
        keys[i] = ((uint64_t)(uint32_t)in_src[in_rp[item_seg(items[i])] + item_round(items[i]) * RT_PER] << 32) |
                  (uint64_t)i;
}

__global__ void k_item_order(int64_t n_items, const uint64_t* __restrict__ keys, const uint64_t* __restrict__ items,
                             uint64_t* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_items; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = items[(uint32_t)keys[i]];
}

// several words into one place, for one copy to the host
struct Words {
    const uint64_t* p[5];
};
__global__ void k_gather_words(Words W, uint64_t* __restrict__ out) {
    if (threadIdx.x < 5) out[threadIdx.x] = *W.p[threadIdx.x];
}

static unsigned plain_blocks(int64_t items) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, (int64_t)device_info().n_cu * 32));
}

void build_in_lists(pg_graph* g, uint64_t* moff_total, uint64_t* heavy_total) {
    MaskPlan& P = g->dag.plan;
    Dag& G = g->dag;
    const int64_t n = g->n, m = G.n_edges;
    const int64_t* rp = G.rp.as<int64_t>();
    const int32_t* col = G.col.as<int32_t>();
    const int32_t* src = G.src.as<int32_t>();
    hipStream_t s = g->stream;
    const bool by_root = m >= DAG_IN_LISTS;
    DevBuf t1, t2;
    Arena ar;
    uint64_t total[5] = {};   // items of each kind, then the sums of the plan's other offsets
    SettleOnError settle(s);
    const int64_t cap = m / WAVE + n + 1;   // items of a class at most
    ar.buf.reserve(sizeof(uint64_t) * (size_t)(256 * ((m + 2047) / 2048) * 3 + 2 * cap + 8 * (n + 1)) + (size_t(8) << 20));
    int bits = 1;
    while ((n >> bits) != 0) ++bits;
    if (by_root) {
        t1.reserve(sizeof(uint64_t) * m);
        t2.reserve(sizeof(uint64_t) * m);
        G.in_edge.reserve(sizeof(int32_t) * m);
        G.in_src.reserve(sizeof(int32_t) * m);
        uint64_t* keys = t1.as<uint64_t>();
        k_in_keys<<<plain_blocks(m), 256, 0, s>>>(n, m, rp, col, src, keys);
        PG_HIP(hipGetLastError());
        radix_sort_u64(keys, t2.as<uint64_t>(), m, 32, 32 + bits, ar, s);
        k_in_rows<<<plain_blocks(n + 1), 256, 0, s>>>(n, m, keys, G.in_rp.as<int64_t>());
        PG_HIP(hipGetLastError());
        k_in_lists<<<plain_blocks(m), 256, 0, s>>>(m, keys, src, G.in_edge.as<int32_t>(), G.in_src.as<int32_t>());
        PG_HIP(hipGetLastError());
    }
    const int64_t* in_rp = G.in_rp.as<int64_t>();
    uint32_t* rounds[3] = {push<uint32_t>(ar, n), push<uint32_t>(ar, n), push<uint32_t>(ar, n)};
    k_in_class<<<plain_blocks(n), 256, 0, s>>>(n, rp, col, in_rp, rounds[RC_TABLE], rounds[RC_LIST], rounds[RC_HASH]);
    PG_HIP(hipGetLastError());
    uint64_t* pos[3];
    for (int c = 0; c < 3; ++c) {
        pos[c] = push<uint64_t>(ar, n + 1);
        scan_u32(rounds[c], n, pos[c], ar, s);
    }
    uint64_t* gathered = push<uint64_t>(ar, 5);
    k_gather_words<<<1, WAVE, 0, s>>>(
        Words{{pos[0] + n, pos[1] + n, pos[2] + n, P.moff.as<uint64_t>() + n, P.hrp.as<uint64_t>() + n}}, gathered);
    PG_HIP(hipGetLastError());
    PG_HIP(hipMemcpyAsync(total, gathered, sizeof(total), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    *moff_total = total[3];
    *heavy_total = total[4];
    for (int c = 0; c < 3; ++c) {
        const int64_t k = P.items[c] = (int64_t)total[c];
        if (k == 0) continue;
        P.item[c].reserve(sizeof(uint64_t) * k);
        const bool sort = c != RC_LIST && by_root;
        uint64_t* items = sort ? push<uint64_t>(ar, k) : P.item[c].as<uint64_t>();
        k_in_items<<<plain_blocks(n), 256, 0, s>>>(n, pos[c], items);
        PG_HIP(hipGetLastError());
        if (sort) {
            // By root: items that run together then read the same lists, out of
            // one die's L2 (in-lists are sorted by root, so RT_PER entries of a
            // long one are of few).
            uint64_t* keys = t1.as<uint64_t>();
            k_item_keys<<<plain_blocks(k), 256, 0, s>>>(k, items, in_rp, G.in_src.as<int32_t>(), keys);
            PG_HIP(hipGetLastError());
            radix_sort_u64(keys, t2.as<uint64_t>(), k, 32, 32 + bits, ar, s);
            k_item_order<<<plain_blocks(k), 256, 0, s>>>(k, keys, items, P.item[c].as<uint64_t>());
            PG_HIP(hipGetLastError());
        }
    }
    PG_HIP(hipStreamSynchronize(s));
}

void count_rows(pg_graph* g, CountArgs A, unsigned long long* queues) {
    const MaskPlan& P = g->dag.plan;
    hipStream_t s = g->stream;
    A.rp = g->dag.rp.as<int64_t>();
    A.col = g->dag.col.as<int32_t>();
    A.moff = P.moff.as<uint64_t>();
    A.in_rp = g->dag.in_rp.as<int64_t>();
    A.in_edge = g->dag.in_edge.as<int32_t>();
    A.in_src = g->dag.in_src.as<int32_t>();
    for (int c = 0; c < 3; ++c) {
        const int64_t n = P.items[c];
        if (n == 0) continue;
        const auto kernel = c == RC_TABLE  ? (A.M ? k_rows_table<true, false> : k_rows_table<false, false>)
                            : c == RC_LIST ? (A.M ? k_rows_list<true> : k_rows_list<false>)
                                           : (A.M ? k_rows_table<true, true> : k_rows_table<false, true>);
        const int takers = c == RC_LIST ? RT_WAVES : 1;   // waves of a workgroup that take items
        const unsigned blocks = queue_blocks(kernel, RT_THREADS, 0, (n + takers - 1) / takers);
        XcdQueue Q;
        Q.next = queues + c * Q_WORDS;
        Q.n_items = n;
        Q.chunk = queue_chunk(n, (int64_t)blocks * takers, c == RC_LIST ? 8 : 1);
        kernel<<<blocks, RT_THREADS, 0, s>>>(Q, P.item[c].as<uint64_t>(), A);
        PG_HIP(hipGetLastError());
    }
}

}  // namespace pg
