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
    int32_t graph;     // index into the caller's id list
    int32_t e_lo, e_hi;  // edge range [e_lo, e_hi) in the graph's (v0 < v1) order
};

struct BatchArgs {
    const int64_t* voff;       // device: vertex offsets of the graphs
    const int64_t* rp;         // global row pointers (positions in col)
    const int32_t* col;        // local ids
    const int64_t* ids;        // graph of each output row
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

// LDS of a workgroup, for graphs of at most n_max vertices: the rows (an odd
// number of 64-bit words apart, so that lanes reading one word of different
// rows spread over the banks), then each vertex's first entry in the graph's
// neighbour lists and its first edge to a larger vertex.
__host__ __device__ constexpr int bt_stride(int W) { return W | 1; }

static size_t bt_lds_bytes(int n_max) {
    const int W = std::max(1, (n_max + 63) / 64);
    return sizeof(uint64_t) * (size_t)n_max * bt_stride(W) + 2 * sizeof(int32_t) * (size_t)(n_max + 1);
}

struct BatchSums {
    uint64_t star = 0, path = 0, cycle = 0, paw = 0, diamond = 0, k4 = 0, tri = 0;
};

constexpr int BT_BCHUNK = 32;   // second vertices of one pair task

// The pair tasks of a graph: (64-vertex block of a, BT_BCHUNK consecutive b)
// with b from the block's start on.  Block x has ceil((n - 64 x) / BT_BCHUNK).
__device__ __forceinline__ int bt_pair_tasks(int n, int x) { return (n - 64 * x + BT_BCHUNK - 1) / BT_BCHUNK; }

// 4-cycles of pair tasks [t_lo, t_hi): a lane holds the row of its a above a
// in registers, and the wave walks b, whose row every lane reads from the
// same LDS address.  Bound by the issue of two ANDs and two bit counts per
// row word.
template <int NT, int W>
__device__ __forceinline__ uint64_t bt_cycles(const uint64_t* rows, int n, int t_lo, int t_hi) {
    constexpr int SW = bt_stride(W);
    uint64_t total = 0;
    int x = 0, first = 0;   // block x holds tasks first ..
    for (int t = t_lo + uniform((int)threadIdx.x / WAVE); t < t_hi; t += NT / WAVE) {
        while (t >= first + bt_pair_tasks(n, x)) first += bt_pair_tasks(n, x++);
        const int a = 64 * x + lane();
        uint64_t ra[W];
#pragma unroll
        for (int y = 0; y < W; ++y) ra[y] = (a < n && y >= x) ? rows[a * SW + y] & above_mask(y, a) : 0ull;
        const int b0 = uniform(64 * x + (t - first) * BT_BCHUNK);
        const int b1 = min(b0 + BT_BCHUNK, n);
        // counts are at most 512, so a task's sums fit 32 bits
        uint32_t s2 = 0, s1 = 0;
        for (int b = b0; b < b1; ++b) {
            const uint64_t* rb = rows + b * SW;
            uint32_t c = 0;
#pragma unroll
            for (int y = 0; y < W; ++y)
                if (y >= x) c += (uint32_t)__popcll(ra[y] & rb[y]);
            c = b > a ? c : 0u;
            s2 += c * c;
            s1 += c;
        }
        total += (uint64_t)((s2 - s1) / 2);
    }
    return total;
}

// Edges [e_lo, e_hi) of the graph, a lane each: triangles, paws, diamonds,
// 4-cliques and paths.  The common neighbours above both ends are taken in
// increasing order; those left over, ANDed with the row of the one taken,
// are the 4-cliques it closes.
template <int NT, int W, bool K4>
__device__ __forceinline__ void bt_edges(const uint64_t* rows, const int32_t* rpl, const int32_t* up,
                                         const int32_t* __restrict__ col, int n, int e_lo, int e_hi, BatchSums& S) {
    constexpr int SW = bt_stride(W);
    // ends of edge e: a holds e in its upper range, b is that neighbour
    auto ends = [&](int e, int& a, int& b) {
        int at = 0, cnt = n;
        while (cnt > 1) {
            const int half = cnt >> 1;
            if (up[at + half] <= e) at += half;
            cnt -= half;
        }
        a = at;
        b = col[rpl[at + 1] - (up[at + 1] - e)];
    };
    int e = e_lo + (int)threadIdx.x;
    int na = 0, nb = 0;
    if (e < e_hi) ends(e, na, nb);
    for (; e < e_hi; e += NT) {
        const int a = na, b = nb;
        if (e + NT < e_hi) ends(e + NT, na, nb);   // the next edge's loads fly during this one
        uint64_t c[W];
        uint32_t t = 0;
#pragma unroll
        for (int y = 0; y < W; ++y) {
            c[y] = rows[a * SW + y] & rows[b * SW + y];
            if (K4) t += (uint32_t)__popcll(c[y]);
            c[y] &= above_mask(y, b);
        }
        if (!K4) {
            uint32_t up_t = 0;
#pragma unroll
            for (int y = 0; y < W; ++y) up_t += (uint32_t)__popcll(c[y]);
            S.tri += up_t;
            continue;
        }
        const uint32_t da = (uint32_t)(rpl[a + 1] - rpl[a]), db = (uint32_t)(rpl[b + 1] - rpl[b]);
        S.path += (uint64_t)(da - 1) * (db - 1);
        S.diamond += (uint64_t)t * (t - 1) / 2;
        uint32_t nt = 0, dsum = 0, k4 = 0;
#pragma unroll
        for (int y = 0; y < W; ++y) {
            uint64_t left = c[y];
            while (left) {
                const int v = y * 64 + __ffsll((unsigned long long)left) - 1;
                left &= left - 1;
                const uint64_t* rv = rows + v * SW;
                k4 += (uint32_t)__popcll(left & rv[y]);
#pragma unroll
                for (int z = y + 1; z < W; ++z) k4 += (uint32_t)__popcll(c[z] & rv[z]);
                dsum += (uint32_t)(rpl[v + 1] - rpl[v]);
                nt++;
            }
        }
        S.tri += nt;
        S.paw += (uint64_t)dsum + (uint64_t)nt * (da + db) - 6ull * nt;
        S.k4 += k4;
    }
}

// One graph item per workgroup.  10,000 graphs of 10..400 vertices and
// densities 0.02..0.3 take 1.35 ms; walking every connected 3-set and
// classifying its candidates by eight masks per row word took 87 ms.
// Bound by LDS reads and vector issue of the triangle loop (lanes whose
// edges have fewer common neighbours wait for the others).
template <int NT>
__global__ __launch_bounds__(NT) void k_batch_motifs(BatchArgs A) {
    extern __shared__ uint64_t bt_lds[];
    __shared__ int32_t s_item;
    __shared__ int32_t wave_tot[NT / WAVE];
    uint64_t* rows = bt_lds;
    int32_t* rpl = reinterpret_cast<int32_t*>(bt_lds + (size_t)A.n_max * bt_stride(max(1, (A.n_max + 63) / 64)));
    int32_t* up = rpl + A.n_max + 1;
    const int64_t n_items = A.n_items_dev ? *A.n_items_dev : A.n_items;
    const int w = threadIdx.x / WAVE;
    while (true) {
        if (threadIdx.x == 0) s_item = (int32_t)min<unsigned long long>(atomicAdd(A.next, 1ull), (unsigned long long)INT32_MAX);
        __syncthreads();
        const int64_t it = uniform(s_item);
        if (it >= n_items) break;
        const BatchItem I = A.items[it];
        const int64_t g = A.ids[I.graph];
        const int64_t v0g = A.voff[g];
        const int n = uniform((int32_t)(A.voff[g + 1] - v0g));
        const int W = (n + 63) / 64;
        const int SW = bt_stride(W);
        const int64_t* rp = A.rp + v0g;
        const int64_t base = rp[0];
        const int32_t* col = A.col + base;
        for (int i = threadIdx.x; i < n * SW; i += NT) rows[i] = 0ull;
        for (int v = threadIdx.x; v <= n; v += NT) rpl[v] = (int32_t)(rp[v] - base);
        __syncthreads();
        // adjacency rows as bitsets, 16 lanes per row
        {
            constexpr int G = 16;
            for (int v = threadIdx.x / G; v < n; v += NT / G) {
                uint32_t* row = reinterpret_cast<uint32_t*>(rows + v * SW);
                const int j1 = rpl[v + 1];
                for (int j = rpl[v] + (int)(threadIdx.x % G); j < j1; j += G) {
                    const uint32_t u = (uint32_t)col[j];
                    atomicOr(&row[u >> 5], 1u << (u & 31));
                }
            }
        }
        __syncthreads();
        // up: exclusive prefix over vertices of their larger neighbours
        {
            int32_t carry = 0;
            for (int c0 = 0; c0 < n; c0 += NT) {
                const int v = c0 + threadIdx.x;
                uint32_t mine = 0;
                if (v < n)
                    for (int y = v >> 6; y < W; ++y) mine += (uint32_t)__popcll(rows[v * SW + y] & above_mask(y, v));
                const uint32_t inc = wave_incl_scan(mine);
                if (lane() == WAVE - 1) wave_tot[w] = (int32_t)inc;
                __syncthreads();
                int32_t before = carry;
                for (int j = 0; j < w; ++j) before += wave_tot[j];
                if (v < n) up[v] = before + (int32_t)(inc - mine);
                for (int j = 0; j < NT / WAVE; ++j) carry += wave_tot[j];
                __syncthreads();
            }
            if (threadIdx.x == 0) up[n] = carry;
        }
        __syncthreads();
        BatchSums S;
        const int E = up[n];
        const int e_lo = uniform(I.e_lo), e_hi = uniform(I.e_hi);
        // vertex sums go with the first part, pair tasks in step with the edges
        if (e_lo == 0) {
            for (int v = threadIdx.x; v < n; v += NT) {
                const uint64_t d = (uint64_t)(rpl[v + 1] - rpl[v]);
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
                bt_edges<NT, WC, false>(rows, rpl, up, col, n, e_lo, e_hi, S);
            } else {
                S.cycle = bt_cycles<NT, WC>(rows, n, t_lo, t_hi);
                bt_edges<NT, WC, true>(rows, rpl, up, col, n, e_lo, e_hi, S);
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
                if (r[c]) atomicAdd(&A.out[(int64_t)I.graph * width + c], (unsigned long long)r[c]);
        __syncthreads();   // the next item overwrites the rows
    }
}

// Validation of every graph of a batch: one wave per vertex (global index);
// entries in [0, n_g), no loop, strictly ascending, reverse entry present.
__global__ __launch_bounds__(256) void k_batch_validate(int64_t n_graphs, const int64_t* __restrict__ voff,
                                                        const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ col, int64_t nnz,
                                                        unsigned* __restrict__ bad_out) {
    const int64_t nv = voff[n_graphs];
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    unsigned bad = 0;
    for (int64_t v = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; v < nv; v += waves) {
        int64_t lo = 0, hi = n_graphs - 1;   // graph of v: last g with voff[g] <= v
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (voff[mid] <= v) lo = mid; else hi = mid - 1;
        }
        const int64_t g0 = voff[lo];
        const int32_t ng = (int32_t)(voff[lo + 1] - g0);
        const int32_t lv = (int32_t)(v - g0);
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        if (r0 < 0 || r1 < r0 || r1 > nnz) { bad |= 1; continue; }
        for (int64_t j = r0 + lane(); j < r1; j += WAVE) {
            const int32_t u = col[j];
            if (u < 0 || u >= ng) { bad |= 2; continue; }
            if (u == lv) bad |= 4;
            if (j > r0 && col[j - 1] >= u) bad |= 8;
            const int64_t q0 = rp[g0 + u], q1 = rp[g0 + u + 1];
            if (q0 < 0 || q1 < q0 || q1 > nnz) continue;
            if (!contains(col + q0, (int32_t)(q1 - q0), lv)) bad |= 16;
        }
    }
    if (bad) atomicOr(bad_out, bad);
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
    DevBuf d_voff, d_rp, d_col, d_all_ids;
    int block_threads = 256;
    double split_work = 4.0e6;
    int grid_blocks = 0;
    int n_max = 0;             // vertices of the largest graph
    int params_gen = 0;        // bumped by pg_batch_set_params; slots re-capture when it moves
    Arena arena;
};

namespace pg {

// Work estimate of a graph: connected 3-vertex subsets (the level-2
// entries) times the row words touched for each.
static double graph_work(int64_t n, int64_t m, const int64_t* rp_local_deg) {
    (void)rp_local_deg;
    if (n <= 0) return 0;
    const double d = 2.0 * (double)m / (double)n;
    const double words = std::ceil((double)n / 64.0);
    return ((double)n * d * d / 2.0 + (double)m) * words + 1.0;
}

static void build_items(pg_batch* b, const int64_t* ids, int64_t n_ids, std::vector<BatchItem>& items,
                        int max_parts = 1 << 20) {
    std::vector<std::pair<double, BatchItem>> tmp;
    tmp.reserve((size_t)n_ids);
    for (int64_t r = 0; r < n_ids; ++r) {
        const int64_t g = ids[r];
        const double w = b->work[(size_t)g];
        const int32_t E = b->n_edges[(size_t)g];
        int parts = (int)std::min<double>(std::max(1.0, std::ceil(w / b->split_work)), std::max(1, E));
        parts = std::min(parts, max_parts);
        for (int p = 0; p < parts; ++p) {
            BatchItem I;
            I.graph = (int32_t)r;
            I.e_lo = (int32_t)((int64_t)E * p / parts);
            I.e_hi = (int32_t)((int64_t)E * (p + 1) / parts);
            tmp.push_back({w / parts, I});
        }
    }
    std::stable_sort(tmp.begin(), tmp.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
    items.resize(tmp.size());
    for (size_t i = 0; i < tmp.size(); ++i) items[i] = tmp[i].second;
}

// Persistent grid of the batch kernel: the tuned size, else as many
// workgroups as a CU's 160 KB of LDS and 16 waves allow (a 512-vertex graph
// takes 41 KB, a 400-vertex one 26 KB); never more workgroups than
// items.
static int batch_grid(const pg_batch* b, int64_t n_items) {
    const int by_lds = (int)((size_t(160) << 10) / (bt_lds_bytes(b->n_max) + 256));
    const int per_cu = std::max(1, std::min(by_lds, 16 * WAVE / b->block_threads));
    const int blocks = b->grid_blocks > 0 ? b->grid_blocks : device_info().n_cu * per_cu;
    return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, n_items));
}

// The launch itself, on a stream that may be capturing.
static void start_batch(const pg_batch* b, const BatchArgs& A, int blocks, hipStream_t s) {
    const size_t lds = bt_lds_bytes(b->n_max);
    switch (b->block_threads) {
        case 64: k_batch_motifs<64><<<blocks, 64, lds, s>>>(A); break;
        case 128: k_batch_motifs<128><<<blocks, 128, lds, s>>>(A); break;
        case 512: k_batch_motifs<512><<<blocks, 512, lds, s>>>(A); break;
        default: k_batch_motifs<256><<<blocks, 256, lds, s>>>(A); break;
    }
}

static void launch_batch(pg_batch* b, int k, const int64_t* d_ids, const BatchItem* d_items, int64_t n_items,
                         uint64_t* d_out, unsigned long long* d_next, hipStream_t s) {
    BatchArgs A;
    A.voff = b->d_voff.as<int64_t>();
    A.rp = b->d_rp.as<int64_t>();
    A.col = b->d_col.as<int32_t>();
    A.ids = d_ids;
    A.items = d_items;
    A.n_items = n_items;
    A.n_items_dev = nullptr;
    A.next = d_next;
    A.out = reinterpret_cast<unsigned long long*>(d_out);
    A.k = k;
    A.n_max = b->n_max;
    fill_u64(reinterpret_cast<uint64_t*>(d_next), 1, 0, s);
    const int blocks = batch_grid(b, n_items);
    ProfScope ps("batch_motifs", s, (double)n_items);
    start_batch(b, A, blocks, s);
    PG_HIP(hipGetLastError());
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
                b->work[(size_t)g] = graph_work(v1 - v0, m2 / 2, nullptr);
            }
            b->d_voff.reserve(sizeof(int64_t) * (n_graphs + 1));
            b->d_rp.reserve(sizeof(int64_t) * (nv + 1));
            b->d_col.reserve(sizeof(int32_t) * std::max<int64_t>(nnz, 1));
            hipStream_t s = b->stream;
            PG_HIP(hipMemcpyAsync(b->d_voff.p, b->voff.data(), sizeof(int64_t) * (n_graphs + 1),
                                  hipMemcpyHostToDevice, s));
            PG_HIP(hipMemcpyAsync(b->d_rp.p, hrp.data(), sizeof(int64_t) * (nv + 1), hipMemcpyHostToDevice, s));
            const hipMemcpyKind ckind = (flags & PG_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
            if (nnz) PG_HIP(hipMemcpyAsync(b->d_col.p, col, sizeof(int32_t) * nnz, ckind, s));
            // identity id list for whole-batch calls
            std::vector<int64_t> all((size_t)std::max<int64_t>(n_graphs, 1));
            std::iota(all.begin(), all.end(), 0);
            b->d_all_ids.reserve(sizeof(int64_t) * all.size());
            PG_HIP(hipMemcpyAsync(b->d_all_ids.p, all.data(), sizeof(int64_t) * all.size(), hipMemcpyHostToDevice, s));
            PG_HIP(hipStreamSynchronize(s));
            // validate every graph on the device: symmetric, sorted, loop-free, in range
            if (nv > 0) {
                DevBuf flag;
                flag.reserve(256);
                fill_u32(flag.as<uint32_t>(), 1, 0, s);
                const int64_t blocks = std::min<int64_t>((nv + 3) / 4, (int64_t)device_info().n_cu * 16);
                k_batch_validate<<<(unsigned)blocks, 256, 0, s>>>(n_graphs, b->d_voff.as<int64_t>(),
                                                                  b->d_rp.as<int64_t>(), b->d_col.as<int32_t>(),
                                                                  nnz, flag.as<unsigned>());
                PG_HIP(hipGetLastError());
                unsigned hf = 0;
                PG_HIP(hipMemcpyAsync(&hf, flag.p, sizeof(hf), hipMemcpyDeviceToHost, s));
                PG_HIP(hipStreamSynchronize(s));
                PG_REQUIRE(hf == 0, PG_EINVAL, "invalid CSR in batch (code " + std::to_string(hf) + ")");
            }
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
            ar.want = std::max<size_t>(ar.want, (size_t)n_ids * (8 + 8 * width) + items.size() * sizeof(BatchItem) + 4096);
            ar.begin_call();
            try {
                int64_t* d_ids = push<int64_t>(ar, n_ids);
                BatchItem* d_items = static_cast<BatchItem*>(ar.push(items.size() * sizeof(BatchItem)));
                uint64_t* d_out = push<uint64_t>(ar, (size_t)n_ids * width);
                unsigned long long* d_next = reinterpret_cast<unsigned long long*>(push<uint64_t>(ar, 1));
                PG_HIP(hipMemcpyAsync(d_ids, ids, sizeof(int64_t) * n_ids, hipMemcpyHostToDevice, s));
                PG_HIP(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, s));
                fill_u64(d_out, (int64_t)n_ids * width, 0, s);
                launch_batch(b, k, d_ids, d_items, (int64_t)items.size(), d_out, d_next, s);
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
// array instead of the batch's arena: the caller's ids, the queue items, the
// output rows and the queue counter.  Each GPU holds its own copy of the
// array (at its own address) until the process ends.  Host code never
// passes the array's name to a kernel or a copy: that name is a host-side
// stand-in, not a device address.  The device address is looked up once per
// device with hipGetSymbolAddress and kept.

namespace pg {

constexpr int64_t NA_MAX_IDS = PG_BATCH_STATIC_MAX_IDS;
constexpr int NA_PARTS = 4;   // queue items per graph at most
constexpr size_t na_align(size_t x) { return (x + 255) & ~size_t(255); }
constexpr size_t NA_IDS = 0;
constexpr size_t NA_ITEMS = NA_IDS + na_align(sizeof(int64_t) * NA_MAX_IDS);
constexpr size_t NA_OUT = NA_ITEMS + na_align(sizeof(BatchItem) * NA_MAX_IDS * NA_PARTS);
constexpr size_t NA_NEXT = NA_OUT + na_align(sizeof(uint64_t) * 6 * NA_MAX_IDS);
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
        build_items(b, ids, n_ids, items, NA_PARTS);
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
        int64_t* d_ids = reinterpret_cast<int64_t*>(base + NA_IDS);
        BatchItem* d_items = reinterpret_cast<BatchItem*>(base + NA_ITEMS);
        uint64_t* d_out = reinterpret_cast<uint64_t*>(base + NA_OUT);
        unsigned long long* d_next = reinterpret_cast<unsigned long long*>(base + NA_NEXT);
        hipStream_t s = b->stream;
        PG_HIP(hipMemcpyAsync(d_ids, ids, sizeof(int64_t) * n_ids, hipMemcpyHostToDevice, s));
        PG_HIP(hipMemcpyAsync(d_items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, s));
        // the array keeps the previous call's rows: clear this call's (a fill
        // kernel); launch_batch clears the queue counter the same way
        fill_u64(d_out, (int64_t)n_ids * width, 0, s);
        launch_batch(b, k, d_ids, d_items, (int64_t)items.size(), d_out, d_next, s);
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
    int64_t* h_ids = nullptr;          // pinned
    BatchItem* h_items = nullptr;      // pinned
    int64_t* h_n = nullptr;            // pinned: number of items
    uint64_t* h_out = nullptr;         // pinned: rows of 6
    DevBuf d_ids, d_items, d_n, d_out, d_next;
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
        if (h_ids) (void)hipHostFree(h_ids);
        if (h_items) (void)hipHostFree(h_items);
        if (h_n) (void)hipHostFree(h_n);
        if (h_out) (void)hipHostFree(h_out);
        if (own_stream && s) (void)hipStreamDestroy(s);
    }
};

namespace pg {

constexpr int SLOT_PARTS = 4;   // queue items per graph at most, in a slot

// Captures one replayable launch: copy ids, items and their number in, clear
// the outputs (fill kernels, no memset nodes), run the persistent kernel,
// copy the rows out.  Buffer sizes are the slot's maxima, so one graph
// serves every submission.
static void capture_slot(pg_batch_slot* S, int k) {
    pg_batch* b = S->b;
    hipStream_t s = S->s;
    const int width = 6;
    BatchArgs A;
    A.voff = b->d_voff.as<int64_t>();
    A.rp = b->d_rp.as<int64_t>();
    A.col = b->d_col.as<int32_t>();
    A.ids = S->d_ids.as<int64_t>();
    A.items = S->d_items.as<BatchItem>();
    A.n_items = 0;
    A.n_items_dev = S->d_n.as<int64_t>();
    A.next = S->d_next.as<unsigned long long>();
    A.out = S->d_out.as<unsigned long long>();
    A.k = k;
    A.n_max = b->n_max;
    // the same grid as a direct launch; the item count is only known on the
    // device, so the slot's maximum bounds it
    const int blocks = batch_grid(b, S->max_items);
    hipGraph_t gr = nullptr;
    PG_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    hipError_t err = hipSuccess;
    do {
        if ((err = hipMemcpyAsync(S->d_ids.p, S->h_ids, sizeof(int64_t) * S->max_ids, hipMemcpyHostToDevice, s))) break;
        if ((err = hipMemcpyAsync(S->d_items.p, S->h_items, sizeof(BatchItem) * S->max_items, hipMemcpyHostToDevice, s))) break;
        if ((err = hipMemcpyAsync(S->d_n.p, S->h_n, sizeof(int64_t), hipMemcpyHostToDevice, s))) break;
        fill_u64(S->d_out.as<uint64_t>(), S->max_ids * width, 0ull, s);
        fill_u64(S->d_next.as<uint64_t>(), 1, 0ull, s);
        start_batch(b, A, blocks, s);
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
            PG_HIP(hipHostMalloc((void**)&S->h_ids, sizeof(int64_t) * max_ids, hipHostMallocDefault));
            PG_HIP(hipHostMalloc((void**)&S->h_items, sizeof(BatchItem) * S->max_items, hipHostMallocDefault));
            PG_HIP(hipHostMalloc((void**)&S->h_n, sizeof(int64_t), hipHostMallocDefault));
            PG_HIP(hipHostMalloc((void**)&S->h_out, sizeof(uint64_t) * max_ids * 6, hipHostMallocDefault));
            std::memset(S->h_ids, 0, sizeof(int64_t) * max_ids);
            std::memset(S->h_items, 0, sizeof(BatchItem) * S->max_items);
            *S->h_n = 0;
            S->d_ids.reserve(sizeof(int64_t) * max_ids);
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
        build_items(S->b, ids, n_ids, items, SLOT_PARTS);
        std::memcpy(S->h_ids, ids, sizeof(int64_t) * n_ids);
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
