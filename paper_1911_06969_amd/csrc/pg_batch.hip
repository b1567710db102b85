// Batched motif counting over many small graphs in one persistent launch
// (the graphs stay resident; a serving loop drives the asynchronous form).
//
// Every graph has at most PG_BATCH_MAX_VERTICES vertices, so a workgroup
// keeps the graph's adjacency as bitset rows in LDS.  The counts of induced
// motifs follow from the numbers of (not necessarily induced) subgraphs of
// each shape, which are sums over pairs and edges of popcounts of row
// intersections:
//   4-cycles    over pairs a < b: C(c, 2), c = common neighbours above a
//               (each cycle at its smallest vertex and the one opposite)
//   diamonds    over edges: C(t, 2), t = common neighbours of the ends
//   paws        over triangles: the degrees of its vertices less 2 each
//   4-cliques   over triangles a < b < c: common neighbours above c
//   paths       over edges: (deg a - 1)(deg b - 1), less 3 per triangle
//   3-stars     over vertices: C(deg, 3)
// Every sum counts each subgraph once, so the sums of a graph's parts add
// up, and the induced counts are whole-number combinations of them: each
// wave converts its own sums (modulo 2^64) and adds them to the output.
// Work items are (graph, range of edges) ordered by estimated work, largest
// first, and taken from an atomic queue by persistent workgroups.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>
#include <type_traits>
#include <vector>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

static_assert(PG_BATCH_MAX_VERTICES <= 512, "rows of at most eight 64-bit words");

struct BatchItem {
    int32_t row;         // output row (index into the caller's id list)
    int32_t graph;
    int32_t e_lo, e_hi;  // edge range [e_lo, e_hi) in the graph's edge list
};

// Where a graph's layout is: its adjacency rows as bitsets (n rows of W =
// ceil(n / 64) words), its vertices' degrees and its edges, ordered by their
// larger end (a | b << 16, a < b).  Laid out once at load time, so that a call
// reads them with coalesced loads alone: building the rows from neighbour
// lists in the counting kernel took a third of its time (430 of 1,180 us on
// 10,000 graphs of 10..400 vertices).
struct BatchGraph {
    int64_t word0;       // first row word (even)
    int64_t edge0;
    int64_t vertex0;
    int32_t n, n_edges;
};

struct BatchArgs {
    const BatchGraph* graphs;
    const uint64_t* rows;
    const uint32_t* edges;
    const uint16_t* deg;
    const BatchItem* items;
    int64_t n_items;
    const int64_t* n_items_dev;   // when set, the item count is read from device memory
    unsigned long long* next;  // queue counter (zeroed before the launch)
    unsigned long long* out;   // rows of 6 (k = 4) or 2 (k = 3)
    int k;
    int n_max;                 // vertices of the batch's largest graph (sizes the LDS)
};

__device__ __forceinline__ uint64_t above_mask(int w, int32_t v) {
    // bits of word w for vertices strictly greater than v
    const int32_t lo = w * 64;
    if (v < lo) return ~0ull;
    if (v >= lo + 63) return 0ull;
    return ~0ull << (v - lo + 1);
}

// First index in [lo, hi) with a[i] > key.
__device__ __forceinline__ int64_t upper_bound64(const int64_t* a, int64_t lo, int64_t hi, int64_t key) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// LDS of a workgroup, for graphs of at most n_max vertices: the rows and
// their upper parts (neighbours above the row's vertex; keeping them saves
// the masks, about 25 instructions per row word and edge), each an odd number
// of 64-bit words apart, so that lanes reading one word of different rows
// spread over the banks, then the degrees.
__host__ __device__ constexpr int bt_stride(int W) { return W | 1; }

static size_t bt_lds_bytes(int n_max) {
    const int W = std::max(1, (n_max + 63) / 64);
    return 2 * sizeof(uint64_t) * (size_t)n_max * bt_stride(W) + sizeof(uint32_t) * (size_t)n_max;
}

struct BatchSums {
    uint64_t star = 0, path = 0, cycle = 0, paw = 0, diamond = 0, k4 = 0, tri = 0;
};

constexpr int BT_BCHUNK = 32;   // second vertices of one pair task

// The pair tasks of a graph: (64-vertex block of a, BT_BCHUNK consecutive b)
// with b from the block's start on.  Block x has ceil((n - 64 x) / BT_BCHUNK).
__device__ __forceinline__ int bt_pair_tasks(int n, int x) { return (n - 64 * x + BT_BCHUNK - 1) / BT_BCHUNK; }

// 4-cycles of one pair task: b in [b0, b1) against the lane's a, whose
// upper row starts at ua (NW words from the block's own word on; lanes past
// the graph repeat its last vertex, which has no b above it).  A b's row is
// read by every lane from the same LDS address, two b at a time.
template <int NW, int SW>
__device__ __forceinline__ uint32_t bt_cycle_task(const uint64_t* ua, const uint64_t* rows, int a, int b0, int b1) {
    uint64_t ra[NW];
#pragma unroll
    for (int y = 0; y < NW; ++y) ra[y] = ua[y];
    uint32_t s2 = 0, s1 = 0;   // counts are at most 512, so a task's sums fit 32 bits
    for (int b = b0; b < b1; b += 2) {
        const uint64_t* rb = rows + b * SW;
        const uint64_t* rc = rows + min(b + 1, b1 - 1) * SW;
        uint32_t c = 0, d = 0;
#pragma unroll
        for (int y = 0; y < NW; ++y) {
            c += (uint32_t)__popcll(ra[y] & rb[y]);
            d += (uint32_t)__popcll(ra[y] & rc[y]);
        }
        c = b > a ? c : 0u;
        d = b + 1 > a && b + 1 < b1 ? d : 0u;
        s2 += c * c + d * d;
        s1 += c + d;
    }
    return (s2 - s1) / 2;
}

// 4-cycles of pair tasks [t_lo, t_hi): a lane holds the row of its a above a
// in registers, and the wave walks b.  Bound by the issue of two ANDs and
// two bit counts per row word.
template <int NT, int W>
__device__ __forceinline__ uint64_t bt_cycles(const uint64_t* rows, const uint64_t* upper, int n, int t_lo, int t_hi) {
    constexpr int SW = bt_stride(W);
    uint64_t total = 0;
    int x = 0, first = 0;   // block x holds tasks first ..
    for (int t = t_lo + uniform((int)threadIdx.x / WAVE); t < t_hi; t += NT / WAVE) {
        while (t >= first + bt_pair_tasks(n, x)) first += bt_pair_tasks(n, x++);
        const int a = min(64 * x + lane(), n - 1);
        const bool own = 64 * x + lane() < n;
        const int b0 = 64 * x + (t - first) * BT_BCHUNK;
        const int b1 = min(b0 + BT_BCHUNK, n);
        const uint64_t* ua = upper + a * SW + x;
        const uint64_t* rx = rows + x;
        uint32_t c = 0;
        switch (W - x) {
            case 1: c = bt_cycle_task<1, SW>(ua, rx, a, b0, b1); break;
            case 2: if constexpr (W >= 2) c = bt_cycle_task<2, SW>(ua, rx, a, b0, b1); break;
            case 3: if constexpr (W >= 3) c = bt_cycle_task<3, SW>(ua, rx, a, b0, b1); break;
            case 4: if constexpr (W >= 4) c = bt_cycle_task<4, SW>(ua, rx, a, b0, b1); break;
            case 5: if constexpr (W >= 5) c = bt_cycle_task<5, SW>(ua, rx, a, b0, b1); break;
            case 6: if constexpr (W >= 6) c = bt_cycle_task<6, SW>(ua, rx, a, b0, b1); break;
            case 7: if constexpr (W >= 7) c = bt_cycle_task<7, SW>(ua, rx, a, b0, b1); break;
            default: if constexpr (W >= 8) c = bt_cycle_task<8, SW>(ua, rx, a, b0, b1); break;
        }
        total += own ? c : 0u;
    }
    return total;
}

// Edges [e_lo, e_hi) of the graph, a lane each: triangles, paws, diamonds,
// 4-cliques and paths.  Edges are numbered by their larger end b, so the
// lanes of a wave mostly share b: one row is a broadcast, and their common
// neighbours above b are of similar number (the triangle loop runs as long
// as its busiest lane).  Each of those, its upper row ANDed with all of them,
// closes the 4-cliques above it.
// The degrees of a triangle's vertices are added up edge by edge: those of
// a and b at its edge (a, b), that of c at its edge (a, c), as common
// neighbours below and above the larger end.
template <int NT, int W, bool K4>
__device__ __forceinline__ void bt_edges(const uint64_t* rows, const uint64_t* upper, const uint32_t* deg,
                                         const uint32_t* __restrict__ edges, int e_lo, int e_hi, BatchSums& S) {
    constexpr int SW = bt_stride(W);
    int e = e_lo + (int)threadIdx.x;
    uint32_t next = e < e_hi ? edges[e] : 0u;
    for (; e < e_hi; e += NT) {
        const int a = (int)(next & 0xffffu), b = (int)(next >> 16);
        if (e + NT < e_hi) next = edges[e + NT];   // flies during this edge
        uint64_t c[W];
        uint32_t t = 0, above = 0, past_a = 0;   // common neighbours: all, above b, above a
#pragma unroll
        for (int y = 0; y < W; ++y) {
            const uint64_t ra = rows[a * SW + y];
            c[y] = ra & upper[b * SW + y];
            above += (uint32_t)__popcll(c[y]);
            if (K4) {
                const uint64_t rb = rows[b * SW + y];
                t += (uint32_t)__popcll(ra & rb);
                past_a += (uint32_t)__popcll(upper[a * SW + y] & rb);
            }
        }
        S.tri += above;
        if (!K4) continue;
        const uint32_t da = deg[a], db = deg[b];
        S.path += (uint64_t)(da - 1) * (db - 1);
        S.diamond += (uint64_t)t * (t - 1) / 2;
        S.paw += (uint64_t)above * (da + db) + (uint64_t)(past_a - above) * db - 6ull * above;
        uint32_t k4 = 0;
#pragma unroll
        for (int y = 0; y < W; ++y) {
            uint64_t left = c[y];
            while (left) {
                const int v = y * 64 + __ffsll((unsigned long long)left) - 1;
                left &= left - 1;
                const uint64_t* rv = upper + v * SW;
#pragma unroll
                for (int z = y; z < W; ++z) k4 += (uint32_t)__popcll(c[z] & rv[z]);
            }
        }
        S.k4 += k4;
    }
}

// One graph item per workgroup.  10,000 graphs of 10..400 vertices and
// densities 0.02..0.3 take 0.76 ms; walking every connected 3-set and
// classifying its candidates by eight masks per row word took 87 ms.
// Bound by the vector issue of the pair and triangle loops (lanes whose
// edges have fewer common neighbours wait for the others).
template <int NT>
__global__ __launch_bounds__(NT) void k_batch_motifs(BatchArgs A) {
    extern __shared__ uint64_t bt_lds[];
    __shared__ int32_t s_item;
    uint64_t* rows = bt_lds;
    const size_t row_words = (size_t)A.n_max * bt_stride(max(1, (A.n_max + 63) / 64));
    uint64_t* upper = bt_lds + row_words;
    uint32_t* deg = reinterpret_cast<uint32_t*>(upper + row_words);
    const int64_t n_items = A.n_items_dev ? *A.n_items_dev : A.n_items;
    while (true) {
        if (threadIdx.x == 0) s_item = (int32_t)min<unsigned long long>(atomicAdd(A.next, 1ull), (unsigned long long)INT32_MAX);
        __syncthreads();
        const int64_t it = uniform(s_item);
        if (it >= n_items) break;
        const BatchItem I = A.items[it];
        const BatchGraph G = A.graphs[uniform(I.graph)];
        const int n = uniform(G.n);
        const int W = (n + 63) / 64;
        const uint32_t* edges = A.edges + uniform64(G.edge0);
        {
            // word i is row v = i / W, word y = i - v W (i < 4096, so the
            // product with the rounded-up reciprocal is exact)
            const uint64_t* src = A.rows + uniform64(G.word0);
            const uint32_t inv = W > 0 ? (65536u + (uint32_t)W - 1) / (uint32_t)W : 0u;
            const int SW = bt_stride(W);
            const int nw = n * W;
            for (int i0 = threadIdx.x; i0 < nw; i0 += 4 * NT) {
                uint64_t r[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) r[q] = src[min(i0 + q * NT, nw - 1)];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + q * NT;
                    if (i < nw) {
                        const int v = (int)(((uint32_t)i * inv) >> 16), y = i - v * W;
                        rows[v * SW + y] = r[q];
                        upper[v * SW + y] = r[q] & above_mask(y, v);
                    }
                }
            }
            for (int v = threadIdx.x; v < n; v += NT) deg[v] = A.deg[G.vertex0 + v];
        }
        __syncthreads();
        BatchSums S;
        const int E = uniform(G.n_edges);
        const int e_lo = uniform(I.e_lo), e_hi = uniform(I.e_hi);
        // vertex sums go with the first part, pair tasks in step with the edges
        if (e_lo == 0) {
            for (int v = threadIdx.x; v < n; v += NT) {
                const uint64_t d = deg[v];
                S.star += A.k == 3 ? d * (d - 1) / 2 : (d >= 2 ? d * (d - 1) * (d - 2) / 6 : 0ull);
            }
        }
        int n_tasks = 0;
        for (int x = 0; x < W; ++x) n_tasks += bt_pair_tasks(n, x);
        const int t_lo = E > 0 ? (int)((int64_t)n_tasks * e_lo / E) : 0;
        const int t_hi = E > 0 ? (int)((int64_t)n_tasks * e_hi / E) : 0;
        auto body = [&](auto wc) {
            constexpr int WC = decltype(wc)::value;
            if (A.k == 3) {
                bt_edges<NT, WC, false>(rows, upper, deg, edges, e_lo, e_hi, S);
            } else {
                S.cycle = bt_cycles<NT, WC>(rows, upper, n, t_lo, t_hi);
                bt_edges<NT, WC, true>(rows, upper, deg, edges, e_lo, e_hi, S);
            }
        };
        switch (W) {
            case 0: break;
            case 1: body(std::integral_constant<int, 1>{}); break;
            case 2: body(std::integral_constant<int, 2>{}); break;
            case 3: body(std::integral_constant<int, 3>{}); break;
            case 4: body(std::integral_constant<int, 4>{}); break;
            case 5: body(std::integral_constant<int, 5>{}); break;
            case 6: body(std::integral_constant<int, 6>{}); break;
            case 7: body(std::integral_constant<int, 7>{}); break;
            default: body(std::integral_constant<int, 8>{}); break;
        }
        // induced counts of this wave's share (modulo 2^64), added once
        const uint64_t star = wave_sum_u64(S.star), tri = wave_sum_u64(S.tri);
        uint64_t r[6] = {0, 0, 0, 0, 0, 0};
        int width = 2;
        if (A.k == 3) {
            r[0] = star - 3 * tri;
            r[1] = tri;
        } else {
            width = 6;
            const uint64_t path = wave_sum_u64(S.path), cycle = wave_sum_u64(S.cycle), paw = wave_sum_u64(S.paw);
            const uint64_t diamond = wave_sum_u64(S.diamond), k4 = wave_sum_u64(S.k4);
            r[5] = k4;
            r[4] = diamond - 6 * k4;
            r[3] = paw - 4 * r[4] - 12 * k4;
            r[2] = cycle - r[4] - 3 * k4;
            r[1] = star - r[3] - 2 * r[4] - 4 * k4;
            r[0] = path - 3 * tri - 2 * r[3] - 4 * r[2] - 6 * r[4] - 12 * k4;
        }
        if (lane() == 0)
            for (int c = 0; c < width; ++c)
                if (r[c]) atomicAdd(&A.out[(int64_t)I.row * width + c], (unsigned long long)r[c]);
        __syncthreads();   // the next item overwrites the rows
    }
}

// The graph of every vertex: the last g with voff[g] <= v.  A search per thread; in the
// passes below, a wave per vertex, it was most of their time.
__global__ void k_batch_graph_of(int64_t nv, int64_t n_graphs, const int64_t* __restrict__ voff,
                                 int32_t* __restrict__ graph_of) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x)
        graph_of[v] = (int32_t)(upper_bound64(voff, 0, n_graphs + 1, v) - 1);
}

// Validation of every graph of a batch: one wave per vertex (global index);
// entries in [0, n_g), no loop, strictly ascending, reverse entry present.  Also each
// vertex's smaller neighbours (the edges it holds).
__global__ __launch_bounds__(256) void k_batch_validate(int64_t nv, const int64_t* __restrict__ voff,
                                                        const int32_t* __restrict__ graph_of,
                                                        const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ col, int64_t nnz,
                                                        uint32_t* __restrict__ low, unsigned* __restrict__ bad_out) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    unsigned bad = 0;
    for (int64_t v = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; v < nv; v += waves) {
        const int32_t g = graph_of[v];
        const int64_t g0 = voff[g];
        const int32_t ng = (int32_t)(voff[g + 1] - g0);
        const int32_t lv = (int32_t)(v - g0);
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        uint32_t less = 0;
        if (r0 < 0 || r1 < r0 || r1 > nnz) {
            bad |= 1;
        } else {
            for (int64_t j = r0 + lane(); j < r1; j += WAVE) {
                const int32_t u = col[j];
                if (u < 0 || u >= ng) { bad |= 2; continue; }
                less += u < lv;
                if (u == lv) bad |= 4;
                if (j > r0 && col[j - 1] >= u) bad |= 8;
                const int64_t q0 = rp[g0 + u], q1 = rp[g0 + u + 1];
                if (q0 < 0 || q1 < q0 || q1 > nnz) continue;
                if (!contains(col + q0, (int32_t)(q1 - q0), lv)) bad |= 16;
            }
        }
        less = wave_sum_u32(less);
        if (lane() == 0) low[v] = less;
    }
    if (bad) atomicOr(bad_out, bad);
}

// Layout: each vertex's row, its degree and the edges it holds.  The CSR is valid by now.
__global__ __launch_bounds__(256) void k_batch_layout(int64_t nv, const int32_t* __restrict__ graph_of,
                                                      const BatchGraph* __restrict__ graphs,
                                                      const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                      const uint64_t* __restrict__ edge_at,
                                                      uint64_t* __restrict__ rows, uint32_t* __restrict__ edges,
                                                      uint16_t* __restrict__ deg) {
    __shared__ uint32_t row[256 / WAVE][PG_BATCH_MAX_VERTICES / 32];
    uint32_t* r = row[threadIdx.x / WAVE];
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    for (int64_t v = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; v < nv; v += waves) {
        const BatchGraph G = graphs[graph_of[v]];
        const uint32_t lv = (uint32_t)(v - G.vertex0);
        const int words = 2 * ((G.n + 63) / 64);   // 32-bit ones
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        const uint64_t e0 = edge_at[v];
        if (lane() < words) r[lane()] = 0u;
        wave_sync();
        for (int64_t j = r0 + lane(); j < r1; j += WAVE) {
            const uint32_t u = (uint32_t)col[j];
            atomicOr(&r[u >> 5], 1u << (u & 31));
            if (u < lv) edges[e0 + (uint64_t)(j - r0)] = u | (lv << 16);
        }
        wave_sync();
        uint32_t* out = reinterpret_cast<uint32_t*>(rows + G.word0) + (int64_t)lv * words;
        if (lane() < words) out[lane()] = r[lane()];
        if (lane() == 0) deg[v] = (uint16_t)(r1 - r0);
        wave_sync();
    }
}

}  // namespace pg

using namespace pg;

struct pg_batch {
    int device = 0;
    hipStream_t stream = nullptr;
    int64_t n_graphs = 0, n_vertices = 0, nnz = 0;
    std::vector<int64_t> voff;     // host copy
    std::vector<int32_t> n_edges;  // per graph
    std::vector<double> work;      // per graph estimate
    DevBuf layout;                 // one block: what follows
    BatchGraph* d_graphs = nullptr;
    uint64_t* d_rows = nullptr;
    uint32_t* d_edges = nullptr;
    uint16_t* d_deg = nullptr;
    int block_threads = 0;     // 0: by the graphs' size
    double split_work = 4.0e6;
    int grid_blocks = 0;
    int n_max = 0;             // vertices of the largest graph
    int params_gen = 0;        // bumped by pg_batch_set_params; slots re-capture when it moves
    Arena arena;
};

namespace pg {

// Work estimate of a graph: connected 3-vertex subsets (the level-2
// entries) times the row words touched for each.
static double graph_work(int64_t n, int64_t m) {
    if (n <= 0) return 0;
    const double d = 2.0 * (double)m / (double)n;
    const double words = std::ceil((double)n / 64.0);
    return ((double)n * d * d / 2.0 + (double)m) * words + 1.0;
}

static int batch_grid(const pg_batch* b, int64_t n_items);
constexpr size_t batch_align(size_t x) { return (x + 255) & ~size_t(255); }

// Work below which a part is not worth its own item: staging a graph takes a
// workgroup about as long as this much counting.
constexpr double BT_MIN_PART = 1.0e5;

// Queue items of graphs ids[0, n_ids), at most max_items (more than n_ids)
// in all, by decreasing estimated work.  A graph is split where its work
// exceeds split_work, or an even share of the call's whole work over the
// workgroups: a call of few graphs would otherwise wait for one workgroup
// with its largest (64 graphs of up to 400 vertices through a slot: 256 us
// with four parts at most, 106 with even shares).
static void build_items(const pg_batch* b, const int64_t* ids, int64_t n_ids, std::vector<BatchItem>& items,
                        int64_t max_items = INT64_MAX) {
    double total = 0;
    for (int64_t r = 0; r < n_ids; ++r) total += b->work[(size_t)ids[r]];
    double part = std::min(b->split_work, std::max(BT_MIN_PART, total / batch_grid(b, INT64_MAX)));
    // sum of ceil(work / part) < total / part + n_ids
    if (max_items < INT64_MAX) part = std::max(part, total / (double)(max_items - n_ids));
    // descending by a counting sort over the leading bits of the estimate
    // (sign and exponent, five bits of mantissa: within 3 %)
    constexpr int BUCKETS = 1 << 13;
    auto parts_of = [&](int64_t g) {
        const double n = std::min(std::max(1.0, std::ceil(b->work[(size_t)g] / part)),
                                  (double)std::max(1, b->n_edges[(size_t)g]));
        return (int64_t)n;
    };
    auto bucket = [&](int64_t g, int64_t parts) {
        const float w = (float)(b->work[(size_t)g] / (double)parts);   // positive
        uint32_t bits;
        std::memcpy(&bits, &w, sizeof(bits));
        return (size_t)(BUCKETS - 1 - (bits >> 18));   // bit 31 is clear
    };
    std::vector<int64_t> at(BUCKETS + 1, 0);
    for (int64_t r = 0; r < n_ids; ++r) {
        const int64_t p = parts_of(ids[r]);
        at[bucket(ids[r], p) + 1] += p;
    }
    for (int i = 0; i < BUCKETS; ++i) at[i + 1] += at[i];
    items.resize((size_t)at[BUCKETS]);
    for (int64_t r = 0; r < n_ids; ++r) {
        const int64_t g = ids[r], parts = parts_of(g), E = b->n_edges[(size_t)g];
        int64_t& o = at[bucket(g, parts)];
        for (int64_t q = 0; q < parts; ++q)
            items[(size_t)o++] = BatchItem{(int32_t)r, (int32_t)g, (int32_t)(E * q / parts),
                                           (int32_t)(E * (q + 1) / parts)};
    }
}

// Workgroups a CU's 160 KB of LDS holds (a 400-vertex graph takes 47 KB, a
// 512-vertex one 76 KB).
static int batch_by_lds(int n_max) { return std::max(1, (int)((size_t(160) << 10) / (bt_lds_bytes(n_max) + 256))); }

// Threads of a workgroup: the tuned number, else 256, or 512 where the LDS
// leaves room for fewer than four workgroups (2,000 graphs of up to 512
// vertices: 325 us with 512 threads, 419 with 256; of up to 64: 121 and 116).
static int batch_threads(int n_max) { return batch_by_lds(n_max) < 4 ? 512 : 256; }
static int batch_threads(const pg_batch* b) { return b->block_threads > 0 ? b->block_threads : batch_threads(b->n_max); }

// Persistent grid of the batch kernel: the tuned size, else as many
// workgroups as a CU's LDS and 16 waves allow (with 32 waves 8,000 graphs of
// up to 64 vertices take longer, drawing items); never more workgroups than
// items.
static int batch_blocks(int n_max, int threads) {
    return device_info().n_cu * std::max(1, std::min(batch_by_lds(n_max), 16 * WAVE / threads));
}
static int batch_grid(const pg_batch* b, int64_t n_items) {
    const int blocks = b->grid_blocks > 0 ? b->grid_blocks : batch_blocks(b->n_max, batch_threads(b));
    return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, n_items));
}

// The launch itself, on a stream that may be capturing.
static void start_batch(int threads, const BatchArgs& A, int blocks, hipStream_t s) {
    const size_t lds = bt_lds_bytes(A.n_max);
    switch (threads) {
        case 64: k_batch_motifs<64><<<blocks, 64, lds, s>>>(A); break;
        case 128: k_batch_motifs<128><<<blocks, 128, lds, s>>>(A); break;
        case 512: k_batch_motifs<512><<<blocks, 512, lds, s>>>(A); break;
        default: k_batch_motifs<256><<<blocks, 256, lds, s>>>(A); break;
    }
}

static BatchArgs batch_args(const pg_batch* b, int k) {
    BatchArgs A{};
    A.graphs = b->d_graphs;
    A.rows = b->d_rows;
    A.edges = b->d_edges;
    A.deg = b->d_deg;
    A.k = k;
    A.n_max = b->n_max;
    return A;
}

static void launch_batch(pg_batch* b, int k, const BatchItem* d_items, int64_t n_items,
                         uint64_t* d_out, unsigned long long* d_next, hipStream_t s) {
    BatchArgs A = batch_args(b, k);
    A.items = d_items;
    A.n_items = n_items;
    A.next = d_next;
    A.out = reinterpret_cast<unsigned long long*>(d_out);
    fill_u64(reinterpret_cast<uint64_t*>(d_next), 1, 0, s);
    const int blocks = batch_grid(b, n_items);
    ProfScope ps("batch_motifs", s, (double)n_items);
    start_batch(batch_threads(b), A, blocks, s);
    PG_HIP(hipGetLastError());
}

// A graph of the size of a batch's as a batch of one, laid out on each call.  The walk
// over two-step paths builds the renamed graph, its plan, the DAG and the clique plan on
// a first call.  First and later calls, by the walk and so: 40 vertices 815, 72 and 50,
// 45 us; 300 of 10 neighbours 844, 76 and 74, 69; K_300 1166, 282 and 170, 163.
__global__ __launch_bounds__(512) void k_batch_low(int n, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                   uint32_t* __restrict__ low) {
    const int v = (int)threadIdx.x;   // low[n, 2 n): the vertices' graph, 0
    if (v >= n) return;
    low[v] = (uint32_t)(lower_bound(col, rp[v], rp[v + 1], v) - rp[v]);
    low[n + v] = 0u;
}

bool count_motifs4_small(pg_graph* g, uint64_t* counts) {
    const int64_t n = g->n, E = g->nnz / 2;
    if (n > PG_BATCH_MAX_VERTICES) return false;
    for (int c = 0; c < 6; ++c) counts[c] = 0;
    if (E == 0) return true;
    hipStream_t s = g->stream;
    Arena& ar = g->arena;
    const int64_t W = (n + 63) / 64;
    const int threads = batch_threads((int)n), most = batch_blocks((int)n, threads);
    const int64_t parts = std::max<int64_t>(
        1, std::min<int64_t>({E, most, (int64_t)(graph_work(n, E) / BT_MIN_PART)}));
    // what the host knows, in one copy: the graph, then the items
    static_assert(sizeof(BatchGraph) % alignof(BatchItem) == 0, "the items follow");
    std::vector<unsigned char> head(sizeof(BatchGraph) + sizeof(BatchItem) * (size_t)parts);
    SettleOnError settle(s);
    const BatchGraph H{0, 0, 0, (int32_t)n, (int32_t)E};
    std::memcpy(head.data(), &H, sizeof(H));
    for (int64_t q = 0; q < parts; ++q) {
        const BatchItem I{0, 0, (int32_t)(E * q / parts), (int32_t)(E * (q + 1) / parts)};
        std::memcpy(head.data() + sizeof(H) + sizeof(I) * (size_t)q, &I, sizeof(I));
    }
    unsigned char* d_head = static_cast<unsigned char*>(ar.push(head.size()));
    uint32_t* low = push<uint32_t>(ar, 2 * n);   // then the vertices' graph, 0
    uint64_t* edge_at = push<uint64_t>(ar, n + 1);
    uint64_t* rows = push<uint64_t>(ar, n * W);
    uint32_t* edges = push<uint32_t>(ar, E);
    uint16_t* deg = push<uint16_t>(ar, n);
    uint64_t* out = push<uint64_t>(ar, 7);   // the counts, then the queue's counter
    PG_HIP(hipMemcpyAsync(d_head, head.data(), head.size(), hipMemcpyHostToDevice, s));
    BatchArgs A{};
    A.graphs = reinterpret_cast<const BatchGraph*>(d_head);
    A.rows = rows;
    A.edges = edges;
    A.deg = deg;
    A.items = reinterpret_cast<const BatchItem*>(d_head + sizeof(BatchGraph));
    A.n_items = parts;
    A.next = reinterpret_cast<unsigned long long*>(out + 6);
    A.out = reinterpret_cast<unsigned long long*>(out);
    A.k = 4;
    A.n_max = (int)n;
    k_batch_low<<<1, 512, 0, s>>>((int)n, g->rp.as<int64_t>(), g->col.as<int32_t>(), low);
    PG_HIP(hipGetLastError());
    scan_u32(low, n, edge_at, ar, s);
    k_batch_layout<<<(unsigned)((n + 3) / 4), 256, 0, s>>>(n, reinterpret_cast<const int32_t*>(low + n), A.graphs,
                                                           g->rp.as<int64_t>(), g->col.as<int32_t>(), edge_at, rows,
                                                           edges, deg);
    PG_HIP(hipGetLastError());
    fill_u64(out, 7, 0, s);
    {
        ProfScope ps("motif_small", s, (double)E);
        start_batch(threads, A, (int)parts, s);
        PG_HIP(hipGetLastError());
    }
    PG_HIP(hipMemcpyAsync(counts, out, sizeof(uint64_t) * 6, hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    return true;
}

}  // namespace pg

namespace pg {
void note_object(int delta);
}

extern "C" {

int pg_batch_load(int64_t n_graphs, const int64_t* voff, const int64_t* row_ptr, const int32_t* col,
                  unsigned flags, void* stream, pg_batch** out) {
    return guarded([&] {
        PG_REQUIRE(out != nullptr && voff != nullptr && row_ptr != nullptr, PG_EINVAL, "NULL argument");
        PG_REQUIRE(n_graphs >= 0 && n_graphs < INT32_MAX, PG_EINVAL, "n_graphs out of range");
        PG_REQUIRE((flags & ~PG_DEVICE_PTRS) == 0, PG_EINVAL, "unknown flag");
        int ndev = 0;
        if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) {
            (void)hipGetLastError();
            throw Error{PG_EDEVICE, "no HIP device available"};
        }
        pg_batch* b = new pg_batch();
        try {
            b->stream = static_cast<hipStream_t>(stream);
            PG_HIP(hipGetDevice(&b->device));
            b->n_graphs = n_graphs;
            b->voff.assign(voff, voff + n_graphs + 1);
            PG_REQUIRE(b->voff[0] == 0, PG_EINVAL, "voff[0] must be 0");
            for (int64_t g = 0; g < n_graphs; ++g) {
                const int64_t n = b->voff[g + 1] - b->voff[g];
                PG_REQUIRE(n >= 0 && n <= PG_BATCH_MAX_VERTICES, PG_EINVAL,
                           "graph " + std::to_string(g) + " has more than PG_BATCH_MAX_VERTICES vertices");
                b->n_max = std::max(b->n_max, (int)n);
            }
            const int64_t nv = b->voff[n_graphs];
            b->n_vertices = nv;
            // row pointers on the host (needed for per-graph edge counts)
            std::vector<int64_t> hrp((size_t)nv + 1);
            const hipMemcpyKind kind = (flags & PG_DEVICE_PTRS) ? hipMemcpyDeviceToHost : hipMemcpyHostToHost;
            PG_HIP(hipMemcpy(hrp.data(), row_ptr, sizeof(int64_t) * (nv + 1), kind));
            const int64_t nnz = hrp[(size_t)nv] - hrp[0];
            PG_REQUIRE(hrp[0] == 0 && nnz >= 0, PG_EINVAL, "row_ptr must start at 0");
            b->nnz = nnz;
            b->n_edges.resize((size_t)n_graphs);
            b->work.resize((size_t)n_graphs);
            for (int64_t g = 0; g < n_graphs; ++g) {
                const int64_t v0 = b->voff[g], v1 = b->voff[g + 1];
                const int64_t m2 = hrp[(size_t)v1] - hrp[(size_t)v0];
                PG_REQUIRE(m2 >= 0 && m2 % 2 == 0, PG_EINVAL, "graph rows not symmetric");
                b->n_edges[(size_t)g] = (int32_t)(m2 / 2);
                b->work[(size_t)g] = graph_work(v1 - v0, m2 / 2);
            }
            hipStream_t s = b->stream;
            std::vector<BatchGraph> graphs((size_t)n_graphs);
            Arena ar;
            SettleOnError settle(s);
            // the CSR on the device and the rest that validation and layout take, in one block
            ar.buf.reserve(sizeof(uint64_t) * (size_t)(n_graphs + 3 * nv + nv / 256 + nnz / 2) + (size_t(1) << 20));
            int64_t* d_voff = push<int64_t>(ar, n_graphs + 1);
            int64_t* d_rp = push<int64_t>(ar, nv + 1);
            int32_t* d_col = push<int32_t>(ar, nnz);
            unsigned* flag = push<unsigned>(ar, 1);
            uint32_t* low = push<uint32_t>(ar, nv);
            int32_t* graph_of = push<int32_t>(ar, nv);
            uint64_t* edge_at = push<uint64_t>(ar, nv + 1);
            PG_HIP(hipMemcpyAsync(d_voff, b->voff.data(), sizeof(int64_t) * (n_graphs + 1),
                                  hipMemcpyHostToDevice, s));
            PG_HIP(hipMemcpyAsync(d_rp, hrp.data(), sizeof(int64_t) * (nv + 1), hipMemcpyHostToDevice, s));
            const hipMemcpyKind ckind = (flags & PG_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
            if (nnz) PG_HIP(hipMemcpyAsync(d_col, col, sizeof(int32_t) * nnz, ckind, s));
            // validate every graph on the device: symmetric, sorted, loop-free, in range
            const int64_t per = (int64_t)device_info().n_cu * 16;
            if (nv > 0) {
                fill_u32(flag, 1, 0, s);
                k_batch_graph_of<<<(unsigned)std::min<int64_t>((nv + 255) / 256, per), 256, 0, s>>>(
                    nv, n_graphs, d_voff, graph_of);
                PG_HIP(hipGetLastError());
                k_batch_validate<<<(unsigned)std::min<int64_t>((nv + 3) / 4, per), 256, 0, s>>>(
                    nv, d_voff, graph_of, d_rp, d_col, nnz, low, flag);
                PG_HIP(hipGetLastError());
                scan_u32(low, nv, edge_at, ar, s);
            }
            // meanwhile the graphs' table
            int64_t words = 0, edges = 0;
            for (int64_t g = 0; g < n_graphs; ++g) {
                const int64_t n = b->voff[g + 1] - b->voff[g];
                graphs[(size_t)g] = BatchGraph{words, edges, b->voff[g], (int32_t)n, b->n_edges[(size_t)g]};
                words += (n * ((n + 63) / 64) + 1) & ~int64_t(1);
                edges += b->n_edges[(size_t)g];
            }
            if (nv > 0) {
                unsigned hf = 0;
                PG_HIP(hipMemcpyAsync(&hf, flag, sizeof(hf), hipMemcpyDeviceToHost, s));
                PG_HIP(hipStreamSynchronize(s));
                PG_REQUIRE(hf == 0, PG_EINVAL, "invalid CSR in batch (code " + std::to_string(hf) + ")");
            }
            // layout
            const size_t at_rows = batch_align(sizeof(BatchGraph) * (size_t)n_graphs);
            const size_t at_edges = at_rows + batch_align(sizeof(uint64_t) * (size_t)words);
            const size_t at_deg = at_edges + batch_align(sizeof(uint32_t) * (size_t)edges);
            b->layout.reserve(at_deg + batch_align(sizeof(uint16_t) * (size_t)nv));
            char* at = b->layout.as<char>();
            b->d_graphs = reinterpret_cast<BatchGraph*>(at);
            b->d_rows = reinterpret_cast<uint64_t*>(at + at_rows);
            b->d_edges = reinterpret_cast<uint32_t*>(at + at_edges);
            b->d_deg = reinterpret_cast<uint16_t*>(at + at_deg);
            // (also where no graph has a vertex: the kernel reads each item's graph)
            if (n_graphs > 0)
                PG_HIP(hipMemcpyAsync(b->d_graphs, graphs.data(), sizeof(BatchGraph) * n_graphs,
                                      hipMemcpyHostToDevice, s));
            if (nv > 0) {
                k_batch_layout<<<(unsigned)std::min<int64_t>((nv + 3) / 4, per), 256, 0, s>>>(
                    nv, graph_of, b->d_graphs, d_rp, d_col, edge_at, b->d_rows, b->d_edges, b->d_deg);
                PG_HIP(hipGetLastError());
            }
            PG_HIP(hipStreamSynchronize(s));   // the buffers above go
            prof_flush();
        } catch (...) {
            delete b;
            throw;
        }
        note_object(1);
        *out = b;
    });
}

int pg_batch_free(pg_batch* b) {
    return guarded([&] {
        if (!b) return;
        (void)hipStreamSynchronize(b->stream);
        delete b;
        note_object(-1);
    });
}

int pg_batch_set_params(pg_batch* b, int block_threads, double split_work, int grid_blocks) {
    return guarded([&] {
        PG_REQUIRE(b != nullptr, PG_EINVAL, "batch is NULL");
        if (block_threads) {
            PG_REQUIRE(block_threads == 64 || block_threads == 128 || block_threads == 256 || block_threads == 512,
                       PG_EINVAL, "block_threads must be 64, 128, 256 or 512");
            b->block_threads = block_threads;
        }
        if (split_work > 0) b->split_work = split_work;
        if (grid_blocks > 0) b->grid_blocks = grid_blocks;
        b->params_gen++;
    });
}

int pg_batch_work_estimate(const pg_batch* b, double* work) {
    return guarded([&] {
        PG_REQUIRE(b != nullptr && work != nullptr, PG_EINVAL, "NULL argument");
        std::memcpy(work, b->work.data(), sizeof(double) * (size_t)b->n_graphs);
    });
}

int pg_batch_count_motifs(pg_batch* b, int k, const int64_t* ids, int64_t n_ids, uint64_t* counts) {
    return guarded([&] {
        PG_REQUIRE(b != nullptr && counts != nullptr, PG_EINVAL, "NULL argument");
        PG_REQUIRE(k == 3 || k == 4, PG_EUNSUPPORTED, "motif size must be 3 or 4");
        std::vector<int64_t> all;
        if (ids == nullptr) {
            n_ids = b->n_graphs;
            all.resize((size_t)n_ids);
            std::iota(all.begin(), all.end(), 0);
            ids = all.data();
        }
        PG_REQUIRE(n_ids >= 0, PG_EINVAL, "n_ids < 0");
        for (int64_t i = 0; i < n_ids; ++i)
            PG_REQUIRE(ids[i] >= 0 && ids[i] < b->n_graphs, PG_EINVAL, "graph id out of range");
        const int width = k == 3 ? 2 : 6;
        if (n_ids == 0) return;
        std::vector<BatchItem> items;
        build_items(b, ids, n_ids, items);
        hipStream_t s = b->stream;
        Arena& ar = b->arena;
        for (int attempt = 0;; ++attempt) {
            ar.want = std::max<size_t>(ar.want, (size_t)n_ids * 8 * width + items.size() * sizeof(BatchItem) + 4096);
            ar.begin_call();
            try {
                BatchItem* d_items = static_cast<BatchItem*>(ar.push(items.size() * sizeof(BatchItem)));
                uint64_t* d_out = push<uint64_t>(ar, (size_t)n_ids * width);
                unsigned long long* d_next = reinterpret_cast<unsigned long long*>(push<uint64_t>(ar, 1));
                PG_HIP(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, s));
                fill_u64(d_out, (int64_t)n_ids * width, 0, s);
                launch_batch(b, k, d_items, (int64_t)items.size(), d_out, d_next, s);
                PG_HIP(hipMemcpyAsync(counts, d_out, sizeof(uint64_t) * n_ids * width, hipMemcpyDeviceToHost, s));
                PG_HIP(hipStreamSynchronize(s));
                prof_flush();
                return;
            } catch (const Error& e) {
                (void)hipStreamSynchronize(s);
                if (e.code == PG_ENOMEM && e.msg == "arena" && attempt < 4) {
                    ar.buf.release();
                    continue;
                }
                throw;
            }
        }
    });
}

}  // extern "C"

// ----------------------------------------------- allocation-free entry point
//
// pg_batch_count_motifs_noalloc keeps its temporaries in one fixed device
// array instead of the batch's arena: the queue items, the output rows and
// the queue counter.  Each GPU holds its own copy of the array (at its own
// address) until the process ends.  Host code never passes the array's name to a kernel or a copy: that name is a host-side
// stand-in, not a device address.  The device address is looked up once per
// device with hipGetSymbolAddress and kept.

namespace pg {

constexpr int64_t NA_MAX_IDS = PG_BATCH_STATIC_MAX_IDS;
constexpr int NA_PARTS = 4;   // queue items at most, per graph on average
constexpr size_t NA_ITEMS = 0;
constexpr size_t NA_OUT = NA_ITEMS + batch_align(sizeof(BatchItem) * NA_MAX_IDS * NA_PARTS);
constexpr size_t NA_NEXT = NA_OUT + batch_align(sizeof(uint64_t) * 6 * NA_MAX_IDS);
constexpr size_t NA_BYTES = NA_NEXT + 256;
static_assert(NA_BYTES <= (size_t(2) << 20), "the allocation-free scratch is 2 MiB at most");

static __device__ __align__(256) unsigned char scratch[NA_BYTES];

constexpr int NA_MAX_DEVICES = 64;
static std::mutex g_na_mu[NA_MAX_DEVICES];
static unsigned char* g_na_ptr[NA_MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up on the
// device's first call); the caller holds g_na_mu[dev].
static unsigned char* scratch_ptr(int dev) {
    if (!g_na_ptr[dev]) {
        void* p = nullptr;
        PG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        PG_REQUIRE(p != nullptr, PG_EDEVICE, "no device address for the static scratch array");
        g_na_ptr[dev] = static_cast<unsigned char*>(p);
    }
    return g_na_ptr[dev];
}

}  // namespace pg

extern "C" {

int pg_batch_count_motifs_noalloc(pg_batch* b, int k, const int64_t* ids, int64_t n_ids, uint64_t* counts) {
    return guarded([&] {
        PG_REQUIRE(b != nullptr && counts != nullptr, PG_EINVAL, "NULL argument");
        PG_REQUIRE(k == 3 || k == 4, PG_EUNSUPPORTED, "motif size must be 3 or 4");
        PG_REQUIRE(b->device >= 0 && b->device < NA_MAX_DEVICES, PG_EDEVICE, "device index out of range");
        std::vector<int64_t> all;
        if (ids == nullptr) {
            n_ids = b->n_graphs;
            all.resize((size_t)n_ids);
            std::iota(all.begin(), all.end(), 0);
            ids = all.data();
        }
        PG_REQUIRE(n_ids >= 0, PG_EINVAL, "n_ids < 0");
        PG_REQUIRE(n_ids <= NA_MAX_IDS, PG_EINVAL,
                   "n_ids exceeds PG_BATCH_STATIC_MAX_IDS (" + std::to_string(NA_MAX_IDS) + ")");
        for (int64_t i = 0; i < n_ids; ++i)
            PG_REQUIRE(ids[i] >= 0 && ids[i] < b->n_graphs, PG_EINVAL, "graph id out of range");
        if (n_ids == 0) return;
        const int width = k == 3 ? 2 : 6;
        std::vector<BatchItem> items;
        build_items(b, ids, n_ids, items, NA_MAX_IDS * NA_PARTS);
        PG_REQUIRE((int64_t)items.size() <= NA_MAX_IDS * NA_PARTS, PG_EINVAL, "too many queue items");

        int prev = 0;
        PG_HIP(hipGetDevice(&prev));
        PG_HIP(hipSetDevice(b->device));
        struct Restore {
            int d;
            ~Restore() { (void)hipSetDevice(d); }
        } restore{prev};
        std::lock_guard<std::mutex> lock(g_na_mu[b->device]);
        unsigned char* base = scratch_ptr(b->device);
        BatchItem* d_items = reinterpret_cast<BatchItem*>(base + NA_ITEMS);
        uint64_t* d_out = reinterpret_cast<uint64_t*>(base + NA_OUT);
        unsigned long long* d_next = reinterpret_cast<unsigned long long*>(base + NA_NEXT);
        hipStream_t s = b->stream;
        PG_HIP(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, s));
        // the array keeps the previous call's rows: clear this call's (a fill
        // kernel); launch_batch clears the queue counter the same way
        fill_u64(d_out, (int64_t)n_ids * width, 0, s);
        launch_batch(b, k, d_items, (int64_t)items.size(), d_out, d_next, s);
        PG_HIP(hipMemcpyAsync(counts, d_out, sizeof(uint64_t) * n_ids * width, hipMemcpyDeviceToHost, s));
        PG_HIP(hipStreamSynchronize(s));
        prof_flush();
    });
}

}  // extern "C"

// ------------------------------------------------------------- slots

struct pg_batch_slot {
    pg_batch* b = nullptr;
    hipStream_t s = nullptr;
    int64_t max_ids = 0, max_items = 0;
    BatchItem* h_items = nullptr;      // pinned
    int64_t* h_n = nullptr;            // pinned: number of items
    uint64_t* h_out = nullptr;         // pinned: rows of 6
    DevBuf d_items, d_n, d_out, d_next;
    hipGraph_t graph[2] = {nullptr, nullptr};          // k = 3, k = 4
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    hipEvent_t done = nullptr;
    bool own_stream = false;           // created here because the caller passed the null stream
    bool pending = false;
    int pending_k = 4;
    int64_t pending_n = 0;
    int params_gen = -1;               // batch parameters the captured graphs were made with
    ~pg_batch_slot() {
        for (int i = 0; i < 2; ++i) {
            if (exec[i]) (void)hipGraphExecDestroy(exec[i]);
            if (graph[i]) (void)hipGraphDestroy(graph[i]);
        }
        if (done) (void)hipEventDestroy(done);
        if (h_items) (void)hipHostFree(h_items);
        if (h_n) (void)hipHostFree(h_n);
        if (h_out) (void)hipHostFree(h_out);
        if (own_stream && s) (void)hipStreamDestroy(s);
    }
};

namespace pg {

constexpr int SLOT_PARTS = 4;   // queue items of a slot, per graph of its capacity

// Captures one replayable launch: copy the items and their number in, clear
// the outputs (fill kernels, no memset nodes), run the persistent kernel,
// copy the rows out.  Buffer sizes are the slot's maxima, so one graph
// serves every submission.
static void capture_slot(pg_batch_slot* S, int k) {
    pg_batch* b = S->b;
    hipStream_t s = S->s;
    const int width = 6;
    BatchArgs A = batch_args(b, k);
    A.items = S->d_items.as<BatchItem>();
    A.n_items_dev = S->d_n.as<int64_t>();
    A.next = S->d_next.as<unsigned long long>();
    A.out = S->d_out.as<unsigned long long>();
    // the same grid as a direct launch; the item count is only known on the
    // device, so the slot's maximum bounds it
    const int blocks = batch_grid(b, S->max_items);
    hipGraph_t gr = nullptr;
    PG_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    hipError_t err = hipSuccess;
    do {
        if ((err = hipMemcpyAsync(S->d_items.p, S->h_items, sizeof(BatchItem) * S->max_items, hipMemcpyHostToDevice, s))) break;
        if ((err = hipMemcpyAsync(S->d_n.p, S->h_n, sizeof(int64_t), hipMemcpyHostToDevice, s))) break;
        fill_u64(S->d_out.as<uint64_t>(), S->max_ids * width, 0ull, s);
        fill_u64(S->d_next.as<uint64_t>(), 1, 0ull, s);
        start_batch(batch_threads(b), A, blocks, s);
        if ((err = hipGetLastError())) break;
        err = hipMemcpyAsync(S->h_out, S->d_out.p, sizeof(uint64_t) * S->max_ids * width, hipMemcpyDeviceToHost, s);
    } while (false);
    hipError_t e2 = hipStreamEndCapture(s, &gr);
    if (err != hipSuccess || e2 != hipSuccess) {
        if (gr) (void)hipGraphDestroy(gr);
        throw Error{PG_EDEVICE, std::string("graph capture failed: ") + hipGetErrorString(err != hipSuccess ? err : e2)};
    }
    hipGraphExec_t ex = nullptr;
    hipError_t e3 = hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0);
    if (e3 != hipSuccess) {
        (void)hipGraphDestroy(gr);
        throw Error{PG_EDEVICE, std::string("graph instantiate failed: ") + hipGetErrorString(e3)};
    }
    if (S->exec[k - 3]) (void)hipGraphExecDestroy(S->exec[k - 3]);
    if (S->graph[k - 3]) (void)hipGraphDestroy(S->graph[k - 3]);
    S->graph[k - 3] = gr;
    S->exec[k - 3] = ex;
}

// (Re)captures both graphs when the batch's parameters changed since the
// last capture; the slot must be idle.
static void ensure_captured(pg_batch_slot* S) {
    if (S->params_gen == S->b->params_gen) return;
    capture_slot(S, 3);
    capture_slot(S, 4);
    S->params_gen = S->b->params_gen;
}

}  // namespace pg

extern "C" {

int pg_batch_slot_create(pg_batch* b, int64_t max_ids, void* stream, pg_batch_slot** out) {
    return guarded([&] {
        PG_REQUIRE(b != nullptr && out != nullptr, PG_EINVAL, "NULL argument");
        PG_REQUIRE(max_ids >= 1 && max_ids <= (int64_t(1) << 24), PG_EINVAL, "max_ids out of range");
        pg_batch_slot* S = new pg_batch_slot();
        try {
            S->b = b;
            S->s = static_cast<hipStream_t>(stream);
            if (S->s == nullptr) {   // the null stream cannot be captured
                PG_HIP(hipStreamCreateWithFlags(&S->s, hipStreamNonBlocking));
                S->own_stream = true;
            }
            S->max_ids = max_ids;
            S->max_items = max_ids * SLOT_PARTS;
            PG_HIP(hipHostMalloc((void**)&S->h_items, sizeof(BatchItem) * S->max_items, hipHostMallocDefault));
            PG_HIP(hipHostMalloc((void**)&S->h_n, sizeof(int64_t), hipHostMallocDefault));
            PG_HIP(hipHostMalloc((void**)&S->h_out, sizeof(uint64_t) * max_ids * 6, hipHostMallocDefault));
            std::memset(S->h_items, 0, sizeof(BatchItem) * S->max_items);
            *S->h_n = 0;
            S->d_items.reserve(sizeof(BatchItem) * S->max_items);
            S->d_n.reserve(sizeof(int64_t));
            S->d_out.reserve(sizeof(uint64_t) * max_ids * 6);
            S->d_next.reserve(sizeof(uint64_t));
            PG_HIP(hipEventCreateWithFlags(&S->done, hipEventDisableTiming));
            ensure_captured(S);
        } catch (...) {
            delete S;
            throw;
        }
        note_object(1);
        *out = S;
    });
}

int pg_batch_slot_submit(pg_batch_slot* S, int k, const int64_t* ids, int64_t n_ids) {
    return guarded([&] {
        PG_REQUIRE(S != nullptr && (ids != nullptr || n_ids == 0), PG_EINVAL, "NULL argument");
        PG_REQUIRE(k == 3 || k == 4, PG_EUNSUPPORTED, "motif size must be 3 or 4");
        PG_REQUIRE(!S->pending, PG_EINVAL, "slot is busy");
        PG_REQUIRE(n_ids >= 0 && n_ids <= S->max_ids, PG_EINVAL, "too many ids for this slot");
        for (int64_t i = 0; i < n_ids; ++i)
            PG_REQUIRE(ids[i] >= 0 && ids[i] < S->b->n_graphs, PG_EINVAL, "graph id out of range");
        ensure_captured(S);   // pg_batch_set_params since the last submission
        std::vector<BatchItem> items;
        build_items(S->b, ids, n_ids, items, S->max_items);
        PG_REQUIRE((int64_t)items.size() <= S->max_items, PG_EINVAL, "too many queue items");
        std::memcpy(S->h_items, items.data(), sizeof(BatchItem) * items.size());
        *S->h_n = (int64_t)items.size();
        PG_HIP(hipGraphLaunch(S->exec[k - 3], S->s));
        PG_HIP(hipEventRecord(S->done, S->s));
        S->pending = true;
        S->pending_k = k;
        S->pending_n = n_ids;
    });
}

int pg_batch_slot_query(pg_batch_slot* S) {
    if (!S) return PG_EINVAL;
    if (!S->pending) return 1;
    hipError_t e = hipEventQuery(S->done);
    if (e == hipSuccess) return 1;
    if (e == hipErrorNotReady) return 0;
    pg::set_error(std::string("hipEventQuery: ") + hipGetErrorString(e));
    return PG_EDEVICE;
}

int pg_batch_slot_wait(pg_batch_slot* S, uint64_t* counts) {
    return guarded([&] {
        PG_REQUIRE(S != nullptr, PG_EINVAL, "slot is NULL");
        if (!S->pending) return;
        PG_HIP(hipEventSynchronize(S->done));
        // the kernel packs rows of the submission's width (2 for k = 3)
        const int width = S->pending_k == 3 ? 2 : 6;
        if (counts) std::memcpy(counts, S->h_out, sizeof(uint64_t) * S->pending_n * width);
        S->pending = false;
    });
}

int pg_batch_slot_free(pg_batch_slot* S) {
    return guarded([&] {
        if (!S) return;
        if (S->pending) (void)hipEventSynchronize(S->done);
        (void)hipStreamSynchronize(S->s);
        delete S;
        note_object(-1);
    });
}

}  // extern "C"
