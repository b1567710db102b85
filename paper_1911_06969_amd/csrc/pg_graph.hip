// Graph ingest: copy, validate on the device, and the derived structures
// the mining pipelines start from (degree-ordered DAG for cliques, the
// single-edge embedding list for motifs).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

enum : unsigned {
    BAD_ROWPTR = 1u,
    BAD_RANGE = 2u,
    BAD_LOOP = 4u,
    BAD_ORDER = 8u,
    BAD_SYMMETRY = 16u,
    BAD_LABEL = 32u,
};

// Passes over all entries take 64 consecutive ones per wave, whatever rows they
// are of: with a wave per row the longest rows held the pass (R-MAT scale 18, edge
// factor 8: 440 us for out-degrees, 67 now), and an entry finds its row by a binary
// search of the row pointers, whose upper levels stay in the caches.
__device__ __forceinline__ int64_t row_of(const int64_t* __restrict__ rp, int64_t n, int64_t j) {
    int64_t lo = 0, hi = n - 1;   // the first row that ends past j
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rp[mid + 1] <= j) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// first lane of each run of equal rows among the lanes, as a mask
__device__ __forceinline__ uint64_t row_heads(int64_t row) {
    const int64_t prev = (int64_t)__shfl_up((long long)row, 1, WAVE);
    return ballot(lane() == 0 || prev != row);
}

// the lanes of the run that starts at lane l
__device__ __forceinline__ uint64_t run_from(uint64_t heads, int l) {
    const uint64_t above = l == WAVE - 1 ? 0ull : heads >> (l + 1) << (l + 1);
    return (above ? (1ull << __builtin_ctzll(above)) - 1ull : ~0ull) & ~((1ull << l) - 1ull);
}

// Sums of a launch on one word: one atomic per workgroup (17 ns each on a line).
constexpr int MAX_BLOCKS = 512;
__device__ __forceinline__ void block_max(uint32_t x, unsigned* out) {
    __shared__ uint32_t m;
    if (threadIdx.x == 0) m = 0u;
    __syncthreads();
    if (x) atomicMax(&m, x);
    __syncthreads();
    if (threadIdx.x == 0 && m) atomicMax(out, m);
}

// Row bounds and labels, and the maximum degree (max_deg[0]: below 2^31, else
// max_deg[1] counts it in units of 2^31).
__global__ __launch_bounds__(256) void k_validate_rows(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ labels, int32_t n_labels,
                                                       unsigned* __restrict__ flags, unsigned* __restrict__ max_deg) {
    unsigned bad = 0;
    uint32_t dlow = 0, dhigh = 0;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        if (v == 0 && r0 != 0) bad |= BAD_ROWPTR;
        if (v == n - 1 && r1 != nnz) bad |= BAD_ROWPTR;
        if (r0 < 0 || r1 < r0 || r1 > nnz) {
            bad |= BAD_ROWPTR;
            continue;
        }
        if (labels && (labels[v] < 0 || labels[v] >= n_labels)) bad |= BAD_LABEL;
        dlow = max(dlow, (uint32_t)min64(r1 - r0, INT32_MAX));
        dhigh = max(dhigh, (uint32_t)((r1 - r0) >> 31));
    }
    if (bad) atomicOr(flags, bad);
    block_max(dlow, max_deg);
    __syncthreads();
    block_max(dhigh, max_deg + 1);
}

// Entries: range; unless bounds_only also no loop, strictly ascending, and the
// reverse entry exists (symmetry).
__device__ __forceinline__ unsigned check_entry(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                const int32_t* __restrict__ col, int64_t v, int64_t r0, int64_t j) {
    const int32_t u = col[j];
    if (u < 0 || u >= n) return BAD_RANGE;
    unsigned bad = 0;
    if (u == v) bad |= BAD_LOOP;
    if (j > r0 && col[j - 1] >= u) bad |= BAD_ORDER;
    const int64_t q0 = rp[u], q1 = rp[u + 1];
    if (q0 < 0 || q1 < q0 || q1 > nnz) return bad;   // reported with u's row
    if (!contains(col + q0, (int32_t)min64(q1 - q0, INT32_MAX), (int32_t)v)) bad |= BAD_SYMMETRY;
    return bad;
}

__global__ __launch_bounds__(256) void k_validate_entries(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                          const int32_t* __restrict__ col, unsigned* __restrict__ flags,
                                                          const unsigned* __restrict__ max_deg, bool bounds_only) {
    unsigned bad = 0;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    const int64_t wave = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE;
    // Rows of 384 entries and more on average, none eight times as long, are taken whole by
    // a wave (2,000 vertices adjacent to 8,000, 32 million entries: 1.35 ms a load, 3.29
    // by entries; 50,000 vertices of 250 neighbours 1.14 and 0.91).  Likewise the sound
    // rows where others are not: the graph is refused already.
    const int64_t most = (int64_t)*(const volatile unsigned*)max_deg;
    const bool by_rows = nnz >= 384 * n && most * n <= 8 * nnz;
    if (by_rows || (*(volatile unsigned*)flags & BAD_ROWPTR)) {
        for (int64_t v = wave; v < n; v += waves) {
            const int64_t r0 = rp[v], r1 = rp[v + 1];
            if (r0 < 0 || r1 < r0 || r1 > nnz) continue;
            for (int64_t j = r0 + lane(); j < r1; j += WAVE) {
                if (bounds_only) bad |= col[j] < 0 || col[j] >= n ? BAD_RANGE : 0u;
                else bad |= check_entry(n, nnz, rp, col, v, r0, j);
            }
        }
    } else {
        for (int64_t j = wave * WAVE + lane(); j < nnz; j += waves * WAVE) {
            if (bounds_only) {
                bad |= col[j] < 0 || col[j] >= n ? BAD_RANGE : 0u;
            } else {
                const int64_t v = row_of(rp, n, j);
                bad |= check_entry(n, nnz, rp, col, v, rp[v], j);
            }
        }
    }
    if (bad) atomicOr(flags, bad);
}

static int bits_for(uint64_t x) {
    int b = 0;
    while (b < 64 && (x >> b) != 0) ++b;
    return b;
}

static unsigned grid_for(int64_t items, int per_block) {
    int64_t b = (items + per_block - 1) / per_block;
    b = std::max<int64_t>(1, std::min<int64_t>(b, (int64_t)device_info().n_cu * 32));
    return (unsigned)b;
}

// ------------------------------------------------------- canonical CSR
//
// PG_CANONICALIZE: the rows are rebuilt as the sorted, duplicate-free,
// loop-free neighbour lists of the symmetric closure: every entry (v, u)
// with u != v gives the keys (v, u) and (u, v), `nb` bits each side by side (a sort
// pass of 8 bits less than by halves for 2^16 to 2^20 vertices); the keys are
// sorted and repeated ones dropped.  Row bounds and vertex ids must be valid already.

constexpr uint64_t NO_EDGE = ~0ull;

__global__ __launch_bounds__(256) void k_canon_keys(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                    const int32_t* __restrict__ col, int nb, uint64_t* __restrict__ keys) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t v = (uint64_t)row_of(rp, n, j);
        const uint64_t u = (uint32_t)col[j];
        const bool loop = u == v;
        keys[2 * j] = loop ? NO_EDGE : (v << nb) | u;
        keys[2 * j + 1] = loop ? NO_EDGE : (u << nb) | v;
    }
}

__global__ void k_canon_keep(int64_t m, const uint64_t* __restrict__ keys, uint32_t* __restrict__ keep) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        keep[i] = (keys[i] != NO_EDGE && (i == 0 || keys[i - 1] != keys[i])) ? 1u : 0u;
}

__global__ void k_canon_write(int64_t m, const uint64_t* __restrict__ keys, const uint32_t* __restrict__ keep,
                              const uint64_t* __restrict__ pos, int nb, int32_t* __restrict__ col) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        if (keep[i]) col[pos[i]] = (int32_t)(keys[i] & ((1ull << nb) - 1ull));
}

// row v starts at the place of the first key of v or above (pos has m + 1 places)
__global__ void k_canon_rows(int64_t n, int64_t m, const uint64_t* __restrict__ keys, const uint64_t* __restrict__ pos,
                             int nb, int64_t* __restrict__ rp) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v <= n; v += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = m;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((keys[mid] >> nb) < (uint64_t)v) lo = mid + 1; else hi = mid;
        }
        rp[v] = (int64_t)pos[lo];
    }
}

static void launch_validate(pg_graph* g, int64_t nnz, const int32_t* labels, int32_t n_labels, unsigned* flags,
                            unsigned* max_deg, bool rows, bool entries, bool bounds_only) {
    hipStream_t s = g->stream;
    const int64_t n = g->n;
    if (n == 0) return;
    if (rows) {
        k_validate_rows<<<std::min(grid_for(n, 256), (unsigned)MAX_BLOCKS), 256, 0, s>>>(
            n, nnz, g->rp.as<int64_t>(), labels, n_labels, flags, max_deg);
        PG_HIP(hipGetLastError());
    }
    if (entries && nnz > 0) {
        k_validate_entries<<<std::min(grid_for(nnz, 256), (unsigned)(device_info().n_cu * 8)), 256, 0, s>>>(
            n, nnz, g->rp.as<int64_t>(), g->col.as<int32_t>(), flags, max_deg, bounds_only);
        PG_HIP(hipGetLastError());
    }
}

static void canonicalize(pg_graph* g) {
    hipStream_t s = g->stream;
    const int64_t n = g->n, nnz = g->nnz;
    DevBuf scratch;
    scratch.reserve(256);
    unsigned* dflags = scratch.as<unsigned>();
    fill_u32(dflags, 4, 0, s);
    launch_validate(g, nnz, nullptr, 0, dflags, dflags + 2, true, true, true);
    unsigned hf = 0;
    PG_HIP(hipMemcpyAsync(&hf, dflags, sizeof(hf), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    if (n == 0 && nnz != 0) hf |= BAD_ROWPTR;
    PG_REQUIRE(hf == 0, PG_EINVAL,
               std::string("invalid CSR (canonicalising needs valid row bounds and vertex ids):") +
                   ((hf & BAD_ROWPTR) ? " row_ptr not monotone or not ending at nnz;" : "") +
                   ((hf & BAD_RANGE) ? " neighbour id out of range;" : ""));
    if (nnz == 0) return;
    const int64_t m = 2 * nnz;
    DevBuf keys, tmp, keep, pos, col2;
    Arena ar;
    SettleOnError settle(s);
    keys.reserve(sizeof(uint64_t) * m);
    tmp.reserve(sizeof(uint64_t) * m);
    keep.reserve(sizeof(uint32_t) * m);
    pos.reserve(sizeof(uint64_t) * (m + 1));
    ar.buf.reserve(sizeof(uint64_t) * (size_t)(256 * ((m + 2047) / 2048) * 3 + (1 << 20)));
    const int nb = std::max(1, bits_for((uint64_t)(n - 1)));
    k_canon_keys<<<grid_for(nnz, 256), 256, 0, s>>>(n, nnz, g->rp.as<int64_t>(), g->col.as<int32_t>(), nb,
                                                    keys.as<uint64_t>());
    PG_HIP(hipGetLastError());
    radix_sort_u64(keys.as<uint64_t>(), tmp.as<uint64_t>(), m, 0, 2 * nb, ar, s);
    k_canon_keep<<<grid_for(m, 256), 256, 0, s>>>(m, keys.as<uint64_t>(), keep.as<uint32_t>());
    PG_HIP(hipGetLastError());
    scan_u32(keep.as<uint32_t>(), m, pos.as<uint64_t>(), ar, s);
    const int64_t nnz2 = (int64_t)read_u64(pos.as<uint64_t>() + m, s);
    col2.reserve(sizeof(int32_t) * std::max<int64_t>(nnz2, 1));
    k_canon_write<<<grid_for(m, 256), 256, 0, s>>>(m, keys.as<uint64_t>(), keep.as<uint32_t>(), pos.as<uint64_t>(),
                                                   nb, col2.as<int32_t>());
    PG_HIP(hipGetLastError());
    k_canon_rows<<<grid_for(n + 1, 256), 256, 0, s>>>(n, m, keys.as<uint64_t>(), pos.as<uint64_t>(), nb,
                                                      g->rp.as<int64_t>());
    PG_HIP(hipGetLastError());
    PG_HIP(hipStreamSynchronize(s));
    std::swap(g->col.p, col2.p);
    std::swap(g->col.bytes, col2.bytes);
    g->nnz = nnz2;
}

void graph_load(pg_graph* g, int64_t n, int64_t nnz, const int64_t* rp, const int32_t* col,
                const int32_t* labels, int32_t n_labels, unsigned flags) {
    PG_REQUIRE(n >= 0 && n < INT32_MAX, PG_EINVAL, "n out of range");
    PG_REQUIRE(nnz >= 0 && nnz < (int64_t(1) << 40), PG_EINVAL, "nnz out of range");
    PG_REQUIRE(rp != nullptr && (col != nullptr || nnz == 0), PG_EINVAL, "null CSR array");
    PG_REQUIRE((labels == nullptr) == (n_labels == 0), PG_EINVAL, "labels and n_labels disagree");
    PG_REQUIRE(n_labels >= 0 && n_labels <= 64, PG_EINVAL, "n_labels must be in [0, 64]");
    hipStream_t s = g->stream;
    g->n = n;
    g->nnz = nnz;
    g->n_labels = n_labels;
    const hipMemcpyKind kind = (flags & PG_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    g->rp.reserve(sizeof(int64_t) * (n + 1));
    g->col.reserve(sizeof(int32_t) * std::max<int64_t>(nnz, 1));
    PG_HIP(hipMemcpyAsync(g->rp.p, rp, sizeof(int64_t) * (n + 1), kind, s));
    if (nnz) PG_HIP(hipMemcpyAsync(g->col.p, col, sizeof(int32_t) * nnz, kind, s));
    if (labels) {
        g->labels.reserve(sizeof(int32_t) * std::max<int64_t>(n, 1));
        if (n) PG_HIP(hipMemcpyAsync(g->labels.p, labels, sizeof(int32_t) * n, kind, s));
    }
    if (flags & PG_CANONICALIZE) {
        canonicalize(g);
        nnz = g->nnz;
    }
    DevBuf scratch;
    scratch.reserve(256);
    unsigned* dflags = scratch.as<unsigned>();   // flags, -, maximum degree (two words)
    fill_u32(dflags, 4, 0, s);
    {
        ProfScope ps("validate", s, (double)nnz);
        // rows rebuilt here are in order and symmetric by construction
        launch_validate(g, nnz, labels ? g->labels.as<int32_t>() : nullptr, n_labels, dflags, dflags + 2, true,
                        !(flags & PG_CANONICALIZE), false);
    }
    unsigned hw[4] = {0, 0, 0, 0};
    PG_HIP(hipMemcpyAsync(hw, dflags, sizeof(hw), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    unsigned hf = hw[0];
    prof_flush();
    if (n == 0 && nnz != 0) hf |= BAD_ROWPTR;
    if (hf) {
        std::string why;
        if (hf & BAD_ROWPTR) why += " row_ptr not monotone or not ending at nnz;";
        if (hf & BAD_RANGE) why += " neighbour id out of range;";
        if (hf & BAD_LOOP) why += " self-loop;";
        if (hf & BAD_ORDER) why += " neighbour list not strictly ascending (or duplicate);";
        if (hf & BAD_SYMMETRY) why += " not symmetric;";
        if (hf & BAD_LABEL) why += " label out of range;";
        throw Error{PG_EINVAL, "invalid CSR:" + why};
    }
    g->max_deg = std::max<int64_t>(hw[2], (int64_t)hw[3] << 31);
}

// ------------------------------------------------------------------- DAG
//
// Orientation of section 4.1: an edge points to the endpoint of higher
// degree, ties to the larger vertex id.  Vertices are renamed by their rank
// in that (degree, id) order, so every DAG edge goes from a smaller to a
// larger rank and each out-list is ascending in rank.

__global__ void k_degree_keys(int64_t n, const int64_t* __restrict__ rp, uint64_t* __restrict__ keys) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        keys[v] = ((uint64_t)(rp[v + 1] - rp[v]) << 32) | (uint64_t)v;
}

__global__ void k_rank_of(int64_t n, const uint64_t* __restrict__ sorted, int32_t* __restrict__ rank_of) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x)
        rank_of[(uint32_t)sorted[r]] = (int32_t)r;
}

// out-degree of every vertex, stored at its rank (zeroed before)
__global__ __launch_bounds__(256) void k_dag_outdeg(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                    const int32_t* __restrict__ col,
                                                    const int32_t* __restrict__ rank_of,
                                                    uint32_t* __restrict__ dout_at_rank) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) & ~63ll; j0 < nnz; j0 += step) {
        const int64_t j = j0 + lane();
        int64_t v = -1;
        int32_t rv = 0;
        bool out = false;
        if (j < nnz) {
            v = row_of(rp, n, j);
            rv = rank_of[v];
            out = rank_of[col[j]] > rv;
        }
        const uint64_t heads = row_heads(v), outs = ballot(out);
        if (v >= 0 && ((heads >> lane()) & 1ull)) {
            const uint32_t c = (uint32_t)popc64(outs & run_from(heads, lane()));
            if (c) atomicAdd(&dout_at_rank[rv], c);
        }
    }
}

// in-degrees from degrees and out-degrees, the largest out-degree, and the paths of two
// edges (an in-edge and an out-edge of one vertex)
__global__ __launch_bounds__(256) void k_dag_indeg(int64_t n, const uint64_t* __restrict__ by_degree,
                                                   const uint32_t* __restrict__ dout, uint32_t* __restrict__ din,
                                                   unsigned* __restrict__ max_out,
                                                   unsigned long long* __restrict__ two_steps) {
    uint32_t mx = 0;
    uint64_t paths = 0;
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t in = (uint32_t)(by_degree[r] >> 32) - dout[r];
        din[r] = in;
        mx = max(mx, dout[r]);
        paths += (uint64_t)in * dout[r];
    }
    block_max(mx, max_out);
    paths = wave_sum_u64(paths);
    __shared__ unsigned long long total;
    if (threadIdx.x == 0) total = 0ull;
    __syncthreads();
    if (lane() == 0 && paths) atomicAdd(&total, (unsigned long long)paths);
    __syncthreads();
    if (threadIdx.x == 0 && total) atomicAdd(two_steps, total);
}

// Every DAG edge (w, v) in the order of rank(v): in_rp[r] = where the in-edges of
// rank r start, taken[r] (zeroed) = how many are placed.  Those of one vertex come in
// any order (no two are of the same w), so a stable sort by w alone leaves each
// out-list ascending.  The key is (rank(w) << 32 | rank(v)), or with head given the
// place in this order instead of rank(v), which goes to head.
__global__ __launch_bounds__(256) void k_dag_emit(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                  const int32_t* __restrict__ col,
                                                  const int32_t* __restrict__ rank_of,
                                                  const int64_t* __restrict__ in_rp, uint32_t* __restrict__ taken,
                                                  uint64_t* __restrict__ keys, int32_t* __restrict__ head_of) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) & ~63ll; j0 < nnz; j0 += step) {
        const int64_t j = j0 + lane();
        int64_t v = -1;
        int32_t rv = 0, rw = 0;
        bool in = false;
        if (j < nnz) {
            v = row_of(rp, n, j);
            rv = rank_of[v];
            rw = rank_of[col[j]];
            in = rw < rv;
        }
        const uint64_t heads = row_heads(v), ins = ballot(in);
        const int head = 63 - __clzll(heads & (lanemask_lt() | (1ull << lane())));
        const uint64_t run = ins & run_from(heads, head);
        int64_t at = 0;
        if (lane() == head && run) at = in_rp[rv] + atomicAdd(&taken[rv], (uint32_t)popc64(run));
        at = (int64_t)__shfl((long long)at, head, WAVE) + popc64(run & lanemask_lt());
        if (in) {
            keys[at] = ((uint64_t)(uint32_t)rw << 32) | (uint64_t)(uint32_t)(head_of ? (int32_t)at : rv);
            if (head_of) head_of[at] = rv;
        }
    }
}

// The sorted (tail << 32 | place in the order of heads): the DAG's edges, and the
// in-lists (the edges in that order).
__global__ void k_dag_lists(int64_t m, const uint64_t* __restrict__ keys, const int32_t* __restrict__ head_of,
                            int32_t* __restrict__ col, int32_t* __restrict__ src, int32_t* __restrict__ in_edge,
                            int32_t* __restrict__ in_src) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[e];
        const uint32_t at = (uint32_t)k;
        col[e] = head_of[at];
        src[e] = (int32_t)(k >> 32);
        in_edge[at] = (int32_t)e;
        in_src[at] = (int32_t)(k >> 32);
    }
}

__global__ void k_split_low(int64_t m, const uint64_t* __restrict__ keys, int32_t* __restrict__ low,
                            int32_t* __restrict__ high) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        low[i] = (int32_t)(uint32_t)keys[i];
        high[i] = (int32_t)(uint32_t)(keys[i] >> 32);
    }
}

void build_dag(pg_graph* g) {
    if (g->dag.built) return;
    hipStream_t s = g->stream;
    const int64_t n = g->n;
    Dag& D = g->dag;
    const int64_t m = g->nnz / 2;
    D.rank_of.reserve(sizeof(int32_t) * std::max<int64_t>(n, 1));
    D.rp.reserve(sizeof(int64_t) * (n + 1));
    D.col.reserve(sizeof(int32_t) * (m + WAVE));   // a wave reads 64 from any place
    D.src.reserve(sizeof(int32_t) * std::max<int64_t>(m, 1));
    DevBuf t1, t2, t3, t4;
    Arena tmp;
    SettleOnError settle(s);
    t1.reserve(sizeof(uint64_t) * std::max<int64_t>(std::max(n, m), 1));
    t2.reserve(sizeof(uint64_t) * std::max<int64_t>(std::max(n, m), 1));
    t3.reserve(sizeof(uint32_t) * std::max<int64_t>(n, 1) + 512);
    t4.reserve(sizeof(uint32_t) * std::max<int64_t>(n, 1));
    tmp.buf.reserve(sizeof(uint64_t) * (size_t)(256 * ((std::max(n, m) + 2047) / 2048) * 3 + (m < DAG_IN_LISTS ? m : 0) + (1 << 20)));
    ProfScope ps("dag_build", s, (double)g->nnz);
    if (n > 0) {
        // 1. degree order: stable sort of (deg << 32 | v) on the degree bits
        uint64_t* keys = t1.as<uint64_t>();
        k_degree_keys<<<grid_for(n, 256), 256, 0, s>>>(n, g->rp.as<int64_t>(), keys);
        PG_HIP(hipGetLastError());
        const int db = std::max(1, bits_for((uint64_t)g->max_deg));
        radix_sort_u64(keys, t2.as<uint64_t>(), n, 32, 32 + db, tmp, s);
        k_rank_of<<<grid_for(n, 256), 256, 0, s>>>(n, keys, D.rank_of.as<int32_t>());
        PG_HIP(hipGetLastError());
        // 2. out- and in-degrees at rank positions, then the DAG row pointers
        // and the places of the in-edges
        uint32_t* dout = t3.as<uint32_t>();
        uint32_t* din = t4.as<uint32_t>();
        unsigned* dmo = reinterpret_cast<unsigned*>(t3.as<char>() + ((sizeof(uint32_t) * n + 255) & ~size_t(255)));
        fill_u32(dout, (int64_t)((reinterpret_cast<char*>(dmo) - t3.as<char>()) / sizeof(uint32_t)) + 4, 0, s);
        const unsigned entry_blocks = std::min(grid_for(std::max<int64_t>(g->nnz, 1), 256), (unsigned)(device_info().n_cu * 8));
        k_dag_outdeg<<<entry_blocks, 256, 0, s>>>(n, g->nnz, g->rp.as<int64_t>(), g->col.as<int32_t>(),
                                                  D.rank_of.as<int32_t>(), dout);
        PG_HIP(hipGetLastError());
        k_dag_indeg<<<std::min(grid_for(n, 256), (unsigned)MAX_BLOCKS), 256, 0, s>>>(
            n, keys, dout, din, dmo, reinterpret_cast<unsigned long long*>(dmo + 2));
        PG_HIP(hipGetLastError());
        scan_u32(dout, n, D.rp.as<uint64_t>(), tmp, s);
        // 3. edges as (rank(src), rank(dst)) keys in the order of dst, sorted by src
        if (m > 0) {
            // (few edges: with the in-lists beside, from the same order)
            const bool in_lists = m < DAG_IN_LISTS;
            D.in_rp.reserve(sizeof(int64_t) * (n + 1));
            scan_u32(din, n, D.in_rp.as<uint64_t>(), tmp, s);
            fill_u32(din, n, 0, s);
            uint64_t* ek = t1.as<uint64_t>();
            int32_t* head_of = nullptr;
            if (in_lists) {
                head_of = reinterpret_cast<int32_t*>(push<uint32_t>(tmp, m));
                D.in_edge.reserve(sizeof(int32_t) * m);
                D.in_src.reserve(sizeof(int32_t) * m);
            }
            k_dag_emit<<<entry_blocks, 256, 0, s>>>(n, g->nnz, g->rp.as<int64_t>(), g->col.as<int32_t>(),
                                                    D.rank_of.as<int32_t>(), D.in_rp.as<int64_t>(), din, ek, head_of);
            PG_HIP(hipGetLastError());
            const int nb = std::max(1, bits_for((uint64_t)(n - 1)));
            radix_sort_u64(ek, t2.as<uint64_t>(), m, 32, 32 + nb, tmp, s);
            if (in_lists)
                k_dag_lists<<<grid_for(m, 256), 256, 0, s>>>(m, ek, head_of, D.col.as<int32_t>(), D.src.as<int32_t>(),
                                                             D.in_edge.as<int32_t>(), D.in_src.as<int32_t>());
            else
                k_split_low<<<grid_for(m, 256), 256, 0, s>>>(m, ek, D.col.as<int32_t>(), D.src.as<int32_t>());
            PG_HIP(hipGetLastError());
        }
        uint64_t h[2] = {0, 0};
        PG_HIP(hipMemcpyAsync(h, dmo, sizeof(h), hipMemcpyDeviceToHost, s));
        PG_HIP(hipStreamSynchronize(s));
        D.max_out = (int64_t)(uint32_t)h[0];
        D.two_steps = (double)h[1];
    } else {
        fill_u64(D.rp.as<uint64_t>(), 1, 0, s);
    }
    PG_HIP(hipStreamSynchronize(s));
    D.n_edges = m;
    D.built = true;
}

// ----------------------------------------------------- motif single edges
//
// The initial embedding list of vertex-induced mining (Algorithm 1, Init):
// every edge once, as (v0, v1) with v0 < v1.  Stored as the upper half of
// each adjacency row: segment of v0 = its neighbours larger than v0.

__global__ __launch_bounds__(256) void k_upper_count(int64_t n, const int64_t* __restrict__ rp,
                                                     const int32_t* __restrict__ col,
                                                     uint32_t* __restrict__ cnt) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        cnt[v] = (uint32_t)(r1 - upper_bound(col, r0, r1, (int32_t)v));
    }
}

__global__ __launch_bounds__(256) void k_upper_write(int64_t n, const int64_t* __restrict__ rp,
                                                     const int32_t* __restrict__ col,
                                                     const uint64_t* __restrict__ seg,
                                                     int32_t* __restrict__ src, int32_t* __restrict__ dst) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    for (int64_t v = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; v < n; v += waves) {
        const int64_t r1 = rp[v + 1];
        const int64_t r0 = r1 - (int64_t)(seg[v + 1] - seg[v]);
        for (int64_t j = r0 + lane(); j < r1; j += WAVE) {
            const uint64_t o = seg[v] + (uint64_t)(j - r0);
            src[o] = (int32_t)v;
            dst[o] = col[j];
        }
    }
}

// for every L1 entry (u, v): the first place in v's row past u
__global__ __launch_bounds__(256) void k_upper_rev(int64_t m, const int64_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col, const int32_t* __restrict__ src,
                                                   const int32_t* __restrict__ dst, int32_t* __restrict__ rev) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < m; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = dst[p];
        const int64_t q0 = rp[v];
        rev[p] = (int32_t)(upper_bound(col, q0, rp[v + 1], src[p]) - q0);
    }
}

void build_motif_l1(pg_graph* g, const MotifView& V) {
    MotifL1& L = *V.ml1;
    if (L.built) return;
    hipStream_t s = g->stream;
    const int64_t n = V.n, m = V.nnz / 2;
    L.seg.reserve(sizeof(int64_t) * (n + 1));
    L.src.reserve(sizeof(int32_t) * std::max<int64_t>(m, 1));
    L.dst.reserve(sizeof(int32_t) * std::max<int64_t>(m, 1));
    L.rev.reserve(sizeof(int32_t) * std::max<int64_t>(m, 1));
    DevBuf cnt;
    Arena tmp;
    SettleOnError settle(s);
    cnt.reserve(sizeof(uint32_t) * std::max<int64_t>(n, 1));
    tmp.buf.reserve(sizeof(uint64_t) * (size_t)(2 * ((n + 2047) / 2048) + 64) + (1 << 16));
    if (n > 0) {
        k_upper_count<<<grid_for(n, 256), 256, 0, s>>>(n, V.rp, V.col, cnt.as<uint32_t>());
        PG_HIP(hipGetLastError());
        scan_u32(cnt.as<uint32_t>(), n, L.seg.as<uint64_t>(), tmp, s);
        k_upper_write<<<grid_for(n, 4), 256, 0, s>>>(n, V.rp, V.col, L.seg.as<uint64_t>(), L.src.as<int32_t>(),
                                                     L.dst.as<int32_t>());
        PG_HIP(hipGetLastError());
        if (m > 0) {
            k_upper_rev<<<grid_for(m, 256), 256, 0, s>>>(m, V.rp, V.col, L.src.as<int32_t>(), L.dst.as<int32_t>(),
                                                        L.rev.as<int32_t>());
            PG_HIP(hipGetLastError());
        }
    } else {
        fill_u64(L.seg.as<uint64_t>(), 1, 0, s);
    }
    PG_HIP(hipStreamSynchronize(s));
    L.n_edges = m;
    L.built = true;
}

void build_motif_l1(pg_graph* g) { build_motif_l1(g, motif_view(g, false)); }

// ------------------------------------------------- renamed graph (motifs)
//
// New name of v = its position in the order of decreasing degree, ties by
// increasing id.  Rows are the renamed neighbour lists, ascending.

__global__ void k_desc_degree_keys(int64_t n, const int64_t* __restrict__ rp, uint64_t max_deg,
                                   uint64_t* __restrict__ keys) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        keys[v] = ((max_deg - (uint64_t)(rp[v + 1] - rp[v])) << 32) | (uint64_t)v;
}

// degree of the vertex named r (for the row pointers)
__global__ void k_renamed_degree(int64_t n, const uint64_t* __restrict__ sorted, const int64_t* __restrict__ rp,
                                 uint32_t* __restrict__ deg) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t v = (uint32_t)sorted[r];
        deg[r] = (uint32_t)(rp[v + 1] - rp[v]);
    }
}

// (name(v) << 32 | name(u)) for every directed entry (v, u), in input order
__global__ __launch_bounds__(256) void k_renamed_edges(int64_t n, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ col,
                                                       const int32_t* __restrict__ name,
                                                       uint64_t* __restrict__ keys) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / WAVE);
    for (int64_t v = blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE; v < n; v += waves) {
        const uint64_t hv = (uint64_t)(uint32_t)name[v] << 32;
        for (int64_t j = rp[v] + lane(); j < rp[v + 1]; j += WAVE) keys[j] = hv | (uint32_t)name[col[j]];
    }
}

void build_motif_graph(pg_graph* g) {
    MotifGraph& M = g->mg;
    if (M.built) return;
    hipStream_t s = g->stream;
    const int64_t n = g->n, nnz = g->nnz;
    M.n = n;
    M.nnz = nnz;
    M.max_deg = g->max_deg;
    M.rp.reserve(sizeof(int64_t) * (n + 1));
    // 64 zeroed entries past the end, so a wave may read a whole 64-entry
    // chunk from any list start
    M.col.reserve(sizeof(int32_t) * (nnz + WAVE));
    PG_HIP(hipMemsetAsync(M.col.as<int32_t>() + nnz, 0, sizeof(int32_t) * WAVE, s));
    DevBuf t1, t2, name, deg, hi;
    Arena tmp;
    SettleOnError settle(s);
    const int64_t big = std::max<int64_t>(std::max(n, nnz), 1);
    t1.reserve(sizeof(uint64_t) * big);
    t2.reserve(sizeof(uint64_t) * big);
    name.reserve(sizeof(int32_t) * std::max<int64_t>(n, 1));
    deg.reserve(sizeof(uint32_t) * std::max<int64_t>(n, 1));
    hi.reserve(sizeof(int32_t) * std::max<int64_t>(nnz, 1));
    tmp.buf.reserve(sizeof(uint64_t) * (size_t)(256 * ((big + 2047) / 2048) * 3 + (1 << 20)));
    ProfScope ps("motif_rename", s, (double)nnz);
    if (n > 0) {
        uint64_t* keys = t1.as<uint64_t>();
        k_desc_degree_keys<<<grid_for(n, 256), 256, 0, s>>>(n, g->rp.as<int64_t>(), (uint64_t)g->max_deg, keys);
        PG_HIP(hipGetLastError());
        const int db = std::max(1, bits_for((uint64_t)g->max_deg));
        radix_sort_u64(keys, t2.as<uint64_t>(), n, 32, 32 + db, tmp, s);
        k_rank_of<<<grid_for(n, 256), 256, 0, s>>>(n, keys, name.as<int32_t>());
        PG_HIP(hipGetLastError());
        k_renamed_degree<<<grid_for(n, 256), 256, 0, s>>>(n, keys, g->rp.as<int64_t>(), deg.as<uint32_t>());
        PG_HIP(hipGetLastError());
        scan_u32(deg.as<uint32_t>(), n, M.rp.as<uint64_t>(), tmp, s);
        if (nnz > 0) {
            uint64_t* ek = t1.as<uint64_t>();
            k_renamed_edges<<<grid_for(n, 4), 256, 0, s>>>(n, g->rp.as<int64_t>(), g->col.as<int32_t>(),
                                                           name.as<int32_t>(), ek);
            PG_HIP(hipGetLastError());
            const int nb = std::max(1, bits_for((uint64_t)(n - 1)));
            radix_sort_u64(ek, t2.as<uint64_t>(), nnz, 0, nb, tmp, s);
            radix_sort_u64(ek, t2.as<uint64_t>(), nnz, 32, 32 + nb, tmp, s);
            k_split_low<<<grid_for(nnz, 256), 256, 0, s>>>(nnz, ek, M.col.as<int32_t>(), hi.as<int32_t>());
            PG_HIP(hipGetLastError());
        }
    } else {
        fill_u64(M.rp.as<uint64_t>(), 1, 0, s);
    }
    PG_HIP(hipStreamSynchronize(s));
    M.built = true;
}

MotifView motif_view(pg_graph* g, bool renamed) {
    if (renamed) {
        build_motif_graph(g);
        MotifGraph& M = g->mg;
        return MotifView{M.n, M.nnz, M.max_deg, M.rp.as<int64_t>(), M.col.as<int32_t>(), &M.ml1};
    }
    return MotifView{g->n, g->nnz, g->max_deg, g->rp.as<int64_t>(), g->col.as<int32_t>(), &g->ml1};
}

}  // namespace pg
