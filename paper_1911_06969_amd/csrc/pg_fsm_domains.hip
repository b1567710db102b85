// Frequent patterns of up to three edges from the labels around each vertex
// (Pangolin sections 2.2 and 3.3, FSM Listing: the same supports as extending
// and filtering embeddings level by level).
//
// The minimum-image support of a pattern is the size of its smallest orbit
// domain, and the domain of an orbit is the set of vertices that some
// embedding places there.  Whether vertex v lies in a domain of a pattern of
// at most three edges is decided by the labels within two steps of v, so the
// domains are counted vertex by vertex, without listing embeddings:
//   edge, wedge and star centres  from the labels of v's neighbours, counted
//                                 up to three each (the masks m1, m2, m3: bit
//                                 l set iff at least 1, 2, 3 neighbours have
//                                 label l);
//   wedge and star leaves         from the masks of v's neighbours, less v;
//   path ends, paths' inner       from the masks of the vertices two steps
//   vertices and triangles        away, and which of those are neighbours of v.
// A vertex's label readings of one shape (the labels at the pattern's other
// vertices) form a set, kept as label masks in LDS, so a vertex counts
// once per pattern and orbit.  A frequent pattern's sub-patterns are frequent
// (the support never grows with the pattern), so filtering changes no
// reported support: with three edges, paths go only over neighbours that some
// frequent wedge leads over, and where there are long lists or few edges per pair
// of labels the edges are counted first and wedges and stars take frequent ones
// alone (each rule beside its kernel's launch).
//
// Workgroups take chunks of vertices of one label, which leaves three labels
// to a path's reading: the counters of the chunk (16 bits: a chunk has fewer
// than 2^16 vertices) fit LDS for up to 32 labels, four waves beside them; beyond,
// they are counted in device memory.
//
// Measured on uniform random graphs, against listing every embedding and
// setting its bits in bitmaps (about 1 KB of keys, sorts and atomics moved per
// hundred embeddings): 500,000 vertices, 2 million edges, 16 labels, three
// edges 32.3 -> 1.54 ms; 100,000 vertices, 1 million edges, 29 labels, two
// edges 5.15 -> 0.16 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "pg_device.h"
#include "pg_fsm.h"
#include "pg_internal.h"

namespace pg {

// A vertex and what is known of it from one step away.  M: 32-bit masks up to
// 32 labels (about half the instructions of 64-bit ones), else 64-bit.
template <class M>
struct FdVertex {
    M m1, m2, m3;          // labels of at least 1, 2, 3 neighbours
    int64_t start;         // its neighbours
    int32_t deg, lab;
};

struct FdArgs {
    const int32_t* col;
    const void* info;         // FdVertex<M> of every vertex
    const uint32_t* order;    // vertices by label
    const int4* chunks;       // (label, first, last + 1 in order, unused)
    int L;
    int lg;                   // log2 of the power of two of lanes that holds L
    int waves;                // of a workgroup
    uint64_t sigma;           // the threshold
    // counters, [label of the vertex][...]
    uint32_t *edge, *wc, *wl;           // [l], [a <= b] centre, [c][b] leaf
    uint32_t *sc, *sl;                  // [a][b][c] centre (a <= b <= c), [c][b1][b2] leaf (b1 <= b2)
    uint32_t *pe, *pi, *tr;             // [l1][l2][l3] end, [l0][l2][l3] inner, [b][c] triangle (b <= c)
    const uint64_t* open;               // [l]: labels c of which some wedge of centre c and a leaf l is frequent
};

constexpr int FD_COOP = 1024;   // vertices of at least this degree are taken by the whole workgroup

template <class M>
__device__ __forceinline__ M fd_bit(int l) {
    return (M)1 << l;
}
__device__ __forceinline__ int fd_first(uint32_t m) { return __builtin_ctz(m); }
__device__ __forceinline__ int fd_first(uint64_t m) { return __builtin_ctzll(m); }
__device__ __forceinline__ uint32_t fd_or(uint32_t* p, uint32_t m) { return atomicOr(p, m); }
__device__ __forceinline__ uint64_t fd_or(uint64_t* p, uint64_t m) {
    return (uint64_t)atomicOr(reinterpret_cast<unsigned long long*>(p), (unsigned long long)m);
}

// labels of at least one (two) neighbours when one of label l is left out
template <class M>
__device__ __forceinline__ M fd_less1(const FdVertex<M>& X, int l) {
    return (X.m1 & ~fd_bit<M>(l)) | (X.m2 & fd_bit<M>(l));
}
template <class M>
__device__ __forceinline__ M fd_less2(const FdVertex<M>& X, int l) {
    return (X.m2 & ~fd_bit<M>(l)) | (X.m3 & fd_bit<M>(l));
}
// the labels above l
template <class M>
__device__ __forceinline__ M fd_above(int l) {
    return ~(M)1 << l;
}

// Counters of one chunk: in LDS (16 bits, two per word) or device memory.
template <bool LDS>
struct FdCount {
    uint32_t* p;
    __device__ __forceinline__ void add(int i) const {
        if (LDS) atomicAdd(&p[i >> 1], 1u << ((i & 1) * 16));
        else atomicAdd(&p[i], 1u);
    }
    // add i * L + l for every bit l of m
    template <class M>
    __device__ __forceinline__ void add_mask(int i, int L, M m) const {
        while (m) {
            add(i * L + fd_first(m));
            m &= m - 1;
        }
    }
    // the same for the bits that m adds to the vertex's mask at `at`
    template <class M>
    __device__ __forceinline__ void add_new(M* at, int i, int L, M m) const {
        if (m & ~*at) add_mask(i, L, (M)(m & ~fd_or(at, m)));
    }
    __device__ __forceinline__ void clear(int n) const {
        if (LDS)
            for (int i = threadIdx.x; i < (n + 1) / 2; i += blockDim.x) p[i] = 0u;
    }
    __device__ __forceinline__ void flush(int n, uint32_t* to) const {
        if (LDS)
            for (int i = threadIdx.x; i < (n + 1) / 2; i += blockDim.x) {
                const uint32_t v = p[i];
                if (v & 0xffffu) atomicAdd(&to[2 * i], v & 0xffffu);
                if (v >> 16) atomicAdd(&to[2 * i + 1], v >> 16);
            }
    }
};

// what two parts of a vertex's neighbours make together
template <class M>
__device__ __forceinline__ void fd_merge(M& m1, M& m2, M& m3, M o1, M o2, M o3) {
    m3 |= o3 | (m2 & o1) | (m1 & o2);
    m2 |= o2 | (m1 & o1);
    m1 |= o1;
}

// Masks of every vertex: G lanes share a vertex's neighbours and merge.  Vertices of
// FD_LONG neighbours or more are left to k_fd_long_masks (`list`, *n_list).
constexpr int FD_LONG = 256;
template <class M>
__global__ __launch_bounds__(256) void k_fd_masks(int64_t n, const int64_t* __restrict__ rp,
                                                  const int32_t* __restrict__ col, const int32_t* __restrict__ lab,
                                                  FdVertex<M>* __restrict__ info, int32_t* __restrict__ list,
                                                  uint32_t* __restrict__ n_list) {
    constexpr int G = 8;
    const int64_t groups = (int64_t)gridDim.x * (256 / G);
    for (int64_t v = blockIdx.x * (int64_t)(256 / G) + threadIdx.x / G; v < n; v += groups) {
        M m1 = 0, m2 = 0, m3 = 0;
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        if (r1 - r0 >= FD_LONG) {
            if (threadIdx.x % G == 0) list[atomicAdd(n_list, 1u)] = (int32_t)v;
            continue;
        }
        for (int64_t j = r0 + threadIdx.x % G; j < r1; j += G) {
            const M b = fd_bit<M>(lab[col[j]]);
            m3 |= m2 & b;
            m2 |= m1 & b;
            m1 |= b;
        }
#pragma unroll
        for (int d = 1; d < G; d <<= 1) {
            const M o1 = __shfl_xor(m1, d, WAVE);
            const M o2 = __shfl_xor(m2, d, WAVE);
            const M o3 = __shfl_xor(m3, d, WAVE);
            fd_merge(m1, m2, m3, o1, o2, o3);
        }
        if (threadIdx.x % G == 0) info[v] = FdVertex<M>{m1, m2, m3, r0, (int32_t)(r1 - r0), lab[v]};
    }
}

// The long lists, a workgroup each, eight elements a thread in flight: a hub of 20,000
// neighbours took eight lanes 630 us.
template <class M>
__global__ __launch_bounds__(1024) void k_fd_long_masks(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                        const int32_t* __restrict__ lab, FdVertex<M>* __restrict__ info,
                                                        const int32_t* __restrict__ list,
                                                        const uint32_t* __restrict__ n_list) {
    __shared__ M part[1024 / WAVE][3];
    constexpr int U = 8;
    const int w = threadIdx.x / WAVE;
    const uint32_t items = *n_list;
    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int32_t v = list[it];
        const int64_t r0 = rp[v], r1 = rp[v + 1];
        M m1 = 0, m2 = 0, m3 = 0;
        for (int64_t j = r0 + threadIdx.x; j < r1; j += 1024 * U) {
            int32_t u[U];
#pragma unroll
            for (int q = 0; q < U; ++q) u[q] = col[min64(j + q * 1024, r1 - 1)];
#pragma unroll
            for (int q = 0; q < U; ++q) u[q] = lab[u[q]];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const M b = j + q * 1024 < r1 ? fd_bit<M>(u[q]) : (M)0;
                m3 |= m2 & b;
                m2 |= m1 & b;
                m1 |= b;
            }
        }
#pragma unroll
        for (int d = 1; d < WAVE; d <<= 1) {
            const M o1 = __shfl_xor(m1, d, WAVE);
            const M o2 = __shfl_xor(m2, d, WAVE);
            const M o3 = __shfl_xor(m3, d, WAVE);
            fd_merge(m1, m2, m3, o1, o2, o3);
        }
        if (lane() == 0) {
            part[w][0] = m1;
            part[w][1] = m2;
            part[w][2] = m3;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < 1024 / WAVE; ++i) fd_merge(m1, m2, m3, part[i][0], part[i][1], part[i][2]);
            info[v] = FdVertex<M>{m1, m2, m3, r0, (int32_t)(r1 - r0), lab[v]};
        }
        __syncthreads();   // the next vertex's parts
    }
}

// One vertex is taken by a wave (or, of FD_COOP neighbours or more, by the
// workgroup): `first` and `step` run over its items, sync() joins them.
struct FdTeam {
    bool all;      // the whole workgroup
    int first, step;
    __device__ __forceinline__ void sync() const {
        if (all) __syncthreads();
        else wave_sync();
    }
};

// Walks a chunk's vertices: those of many neighbours by all waves together,
// then the others by a wave each (the next one's masks are loaded ahead).
template <class M, class F>
__device__ __forceinline__ void fd_chunk(const FdArgs& A, const int4& K, int w, F&& f) {
    const FdVertex<M>* info = static_cast<const FdVertex<M>*>(A.info);
    for (int i = K.y; i < K.z; ++i) {
        const int32_t v = (int32_t)A.order[i];
        const FdVertex<M> V = info[v];
        if (V.deg >= FD_COOP) f(v, V, FdTeam{true, (int)threadIdx.x, (int)blockDim.x});
    }
    __syncthreads();
    int i = K.y + w;
    int32_t nv = 0;
    FdVertex<M> nV{};
    if (i < K.z) {
        nv = uniform((int32_t)A.order[i]);
        nV = info[nv];
    }
    for (; i < K.z; i += A.waves) {
        const int32_t v = nv;
        const FdVertex<M> V = nV;
        if (i + A.waves < K.z) {
            nv = uniform((int32_t)A.order[i + A.waves]);
            nV = info[nv];
        }
        if (V.deg < FD_COOP) f(v, V, FdTeam{false, lane(), WAVE});
    }
    __syncthreads();
}

// 64-bit words of n masks
template <class M>
__host__ __device__ constexpr int fd_words(int n) {
    return (int)((sizeof(M) * (size_t)n + 7) / 8);
}

// The labels of m in order (list: LDS of the wave); returns their number.
__device__ __forceinline__ int fd_list(uint64_t m, uint8_t* list) {
    if ((m >> lane()) & 1ull) list[popc64(m & lanemask_lt())] = (uint8_t)lane();
    wave_sync();
    return popc64(m);
}

// i / n for i < n^2, n <= 64: the product with the rounded-up reciprocal is
// exact (its error, below 64 i / 2^20 < 1 / n, never reaches the next quotient).
__device__ __forceinline__ uint32_t fd_inv(int n) { return n > 0 ? ((1u << 20) + (uint32_t)n - 1) / (uint32_t)n : 0u; }
__device__ __forceinline__ int fd_div(int i, uint32_t inv) { return (int)(((uint32_t)i * inv) >> 20); }

// Edges alone, for patterns of one edge and where they filter the wedges and stars: a wave takes a run of chunks,
// 64 vertices at a time; lane l counts those with a neighbour of label l.
template <class M>
__global__ __launch_bounds__(256) void k_fd_edges(FdArgs A, int n_chunks) {
    const FdVertex<M>* info = static_cast<const FdVertex<M>*>(A.info);
    const int waves = (int)(gridDim.x * (blockDim.x / WAVE)), w = (int)(blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE);
    const int last = (int)((int64_t)n_chunks * (w + 1) / waves);
    int c = (int)((int64_t)n_chunks * w / waves), lab = -1;
    uint32_t cnt = 0;
    auto flush = [&]() {
        if (lane() < A.L && cnt) atomicAdd(&A.edge[lab * A.L + lane()], cnt);
        cnt = 0;
    };
    for (; c < last; ++c) {
        const int4 K = A.chunks[c];
        if (uniform(K.x) != lab) {
            flush();
            lab = uniform(K.x);
        }
        for (int i = uniform(K.y); i < uniform(K.z); i += WAVE) {
            const M m = i + lane() < K.z ? info[A.order[i + lane()]].m1 : (M)0;
            for (int l = 0; l < A.L; ++l) {
                const uint32_t x = (uint32_t)popc64(ballot((m >> l) & 1));
                if (lane() == l) cnt += x;
            }
        }
    }
    flush();
}

// Edges, wedges and (STARS) 3-stars; with FILTER, where edges are counted already,
// wedges and stars along frequent edges (the others are infrequent: uncounted, they
// stay below the threshold).
// A mask's new bits are counted by the lane that sets them.  Bound by the latency of a vertex's chain (its masks, its
// neighbours' masks, the LDS readings) at the waves that LDS leaves resident:
// 582 us for 500,000 vertices of 8 neighbours with 3-stars, 111 us for 100,000
// of 20 without (a pass over its neighbours' masks from HBM takes 10 to 20 us).
template <class M, bool STARS, bool FILTER, bool LDS>
__global__ __launch_bounds__(512) void k_fd_stars(FdArgs A) {
    extern __shared__ __align__(16) uint64_t fd_lds[];
    const int L = A.L, L2 = L * L, L3 = L2 * L;
    const int w = uniform((int)threadIdx.x / WAVE);
    const int4 K = A.chunks[blockIdx.x];
    const int lv = K.x;
    M along = ~(M)0;   // labels that v's frequent edges lead to
    if constexpr (FILTER) {
        uint32_t e = 0;
        if (lane() < L) e = min(A.edge[lv * L + lane()], A.edge[lane() * L + lv]);
        along = (M)ballot(e > 0 && e >= A.sigma);
        if (along == 0) return;   // all waves alike
    }
    // leaf masks of a vertex: wedges [c], stars [c][b1]: labels b2 >= b1
    const int masks = (STARS ? L2 : 0) + L;
    const int words = fd_words<M>(masks) + 8;
    M* own = reinterpret_cast<M*>(fd_lds + (size_t)w * words);
    uint8_t* list = reinterpret_cast<uint8_t*>(own + masks);
    const FdVertex<M>* info = static_cast<const FdVertex<M>*>(A.info);
    uint32_t* cp = reinterpret_cast<uint32_t*>(fd_lds + (size_t)A.waves * words);
    FdCount<LDS> ed{A.edge + (int64_t)lv * L}, wc{A.wc + (int64_t)lv * L2}, wl{A.wl + (int64_t)lv * L2};
    FdCount<LDS> sc{STARS ? A.sc + (int64_t)lv * L3 : nullptr}, sl{STARS ? A.sl + (int64_t)lv * L3 : nullptr};
    if (LDS) {
        ed.p = cp;
        wc.p = ed.p + (L + 1) / 2;
        wl.p = wc.p + (L2 + 1) / 2;
        sc.p = wl.p + (L2 + 1) / 2;
        sl.p = sc.p + (L3 + 1) / 2;
    }
    ed.clear(L);
    wc.clear(L2);
    wl.clear(L2);
    if (STARS) {
        sc.clear(L3);
        sl.clear(L3);
    }
    __syncthreads();
    fd_chunk<M>(A, K, w, [&](int32_t v, const FdVertex<M>& V, const FdTeam& T) {
        M* tab = T.all ? reinterpret_cast<M*>(fd_lds) : own;
        M* leaf = tab + L;
        for (int i = T.first; i < masks; i += T.step) tab[i] = 0;
        T.sync();
        // a power of two of lanes, one per label, share a neighbour
        const int lg = STARS ? A.lg : 0;
        const int b = T.first & ((1 << lg) - 1);
        for (int32_t j = T.first >> lg; j < V.deg; j += T.step >> lg) {
            const FdVertex<M> S = info[A.col[V.start + j]];
            if (FILTER && !((along >> S.lab) & 1)) continue;
            const M m1 = fd_less1(S, lv), m2 = fd_less2(S, lv);
            if (b == 0 && (m1 & ~tab[S.lab])) fd_or(&tab[S.lab], m1);
            if (STARS && b < L && ((m1 >> b) & 1))
                sl.add_new(&leaf[S.lab * L + b], S.lab * L + b, L, (M)((m1 & fd_above<M>(b)) | (m2 & fd_bit<M>(b))));
        }
        T.sync();
        for (int i = T.first; i < L << A.lg; i += T.step) {   // wedge leaves: a lane per (centre, label)
            const int c = i >> A.lg, l = i & ((1 << A.lg) - 1);
            if (l < L && ((tab[c] >> l) & 1)) wl.add(c * L + l);
        }
        const M m1 = FILTER ? V.m1 & along : V.m1;
        const int n1 = fd_list((uint64_t)m1, list);
        const uint32_t inv = fd_inv(n1);
        if (T.first < n1) {   // at most 64 labels
            const int a = list[T.first];
            if (!FILTER) ed.add(a);
            wc.add_mask(a, L, (M)((m1 & fd_above<M>(a)) | (V.m2 & fd_bit<M>(a))));
        }
        if (STARS)
            for (int i = T.first; i < n1 * n1; i += T.step) {
                const int q = fd_div(i, inv), a = list[q], b = list[i - q * n1];
                if (b < a) continue;
                M m = 0;
                if (a < b) m = (m1 & fd_above<M>(b)) | (V.m2 & fd_bit<M>(b));
                else if (V.m2 & fd_bit<M>(a)) m = (m1 & fd_above<M>(b)) | (V.m3 & fd_bit<M>(b));
                sc.add_mask(a * L + b, L, m);
            }
        T.sync();   // the next vertex clears the masks
    });
    if (!FILTER) ed.flush(L, A.edge + (int64_t)lv * L);
    wc.flush(L2, A.wc + (int64_t)lv * L2);
    wl.flush(L2, A.wl + (int64_t)lv * L2);
    if (STARS) {
        sc.flush(L3, A.sc + (int64_t)lv * L3);
        sl.flush(L3, A.sl + (int64_t)lv * L3);
    }
}

// Paths of three edges and triangles.
//
// A wave lays the neighbour lists of 64 neighbours w1 of v end to end and
// takes 64 elements x a step.  For each: is x a neighbour of v (a triangle),
// and which labels may end the path v - w1 - x - . (those of x's neighbours
// other than w1 and v).  For paths with v inside, . - v - w2 - ., the two ends
// may be of any available labels unless they would have to be the same
// vertex: one label l with a single such neighbour on both sides, which is
// then a common neighbour of v and w2.
//
// Bound by instructions: 32 million elements x (500,000 vertices of 8
// neighbours) take 830 us, of which the bits of new readings are most.  Laying
// the lists end to end keeps the lanes busy on short lists; a list per step would
// fill 8 of 64.
//
// The Filter of the level pipeline, as far as it saves work: a pattern that holds
// an infrequent wedge v - w1 - x need not be counted (its support stays at or below
// its true one, so below the threshold), and the lists of neighbours w1 that no
// frequent wedge leads over are not walked.
template <class M, bool LDS>
__global__ __launch_bounds__(512) void k_fd_paths(FdArgs A) {
    extern __shared__ __align__(16) uint64_t fd_lds[];
    const int L = A.L, L2 = L * L, L3 = L2 * L;
    const int w = uniform((int)threadIdx.x / WAVE);
    const int4 K = A.chunks[blockIdx.x];
    const int lv = K.x;
    const uint64_t over = A.open[lv];   // labels of the neighbours w1 to go over
    if (over == 0ull) return;
    const M bv = fd_bit<M>(lv);
    const FdVertex<M>* info = static_cast<const FdVertex<M>*>(A.info);
    // per wave: label masks of a vertex (end [l1][l2], inner [l2] and its
    // diagonal, triangle [b]); common labels, list starts, prefix and labels
    // of 64 neighbours
    const int masks = L2 + 3 * L;
    const int words = fd_words<M>(masks + WAVE) + 3 * WAVE + 8;
    M* own = reinterpret_cast<M*>(fd_lds + (size_t)w * words);
    M* common = own + masks;
    int64_t* lo = reinterpret_cast<int64_t*>(fd_lds + (size_t)w * words + fd_words<M>(masks + WAVE));
    uint32_t* pre = reinterpret_cast<uint32_t*>(lo + WAVE);
    int32_t* lab = reinterpret_cast<int32_t*>(pre + WAVE);
    int32_t* near_list = lab + WAVE;   // v's neighbours, when at most 128
    uint8_t* list = reinterpret_cast<uint8_t*>(near_list + 2 * WAVE);
    uint32_t* cp = reinterpret_cast<uint32_t*>(fd_lds + (size_t)A.waves * words);
    FdCount<LDS> pe{A.pe + (int64_t)lv * L3}, pi{A.pi + (int64_t)lv * L3}, tr{A.tr + (int64_t)lv * L2};
    if (LDS) {
        pe.p = cp;
        pi.p = pe.p + (L3 + 1) / 2;
        tr.p = pi.p + (L3 + 1) / 2;
    }
    pe.clear(L3);
    pi.clear(L3);
    tr.clear(L2);
    __syncthreads();
    fd_chunk<M>(A, K, w, [&](int32_t v, const FdVertex<M>& V, const FdTeam& T) {
        M* tab = T.all ? reinterpret_cast<M*>(fd_lds) : own;
        M* inner = tab + L2;
        M* diag = inner + L;
        M* tri = diag + L;
        for (int i = T.first; i < masks; i += T.step) tab[i] = 0;
        const int64_t r0 = V.start;
        const int32_t d = V.deg;
        const bool staged = d <= 2 * WAVE;
        if (staged)
            for (int i = lane(); i < d; i += WAVE) near_list[i] = A.col[r0 + i];
        T.sync();
        for (int32_t c0 = T.all ? w * WAVE : 0; c0 < d; c0 += T.step) {
            const int nx = min(WAVE, d - c0);
            FdVertex<M> W{};
            bool on = false;
            if (lane() < nx) {
                W = info[staged ? near_list[c0 + lane()] : A.col[r0 + c0 + lane()]];
                lo[lane()] = W.start;
                lab[lane()] = W.lab;
                on = (over >> W.lab) & 1ull;
            }
            common[lane()] = 0;
            const uint32_t len = on ? (uint32_t)W.deg : 0u;
            const uint32_t inc = wave_incl_scan(len);
            pre[lane()] = inc - len;
            const uint32_t total = bcast(inc, WAVE - 1);
            wave_sync();
            for (uint32_t t = lane(); t < total; t += WAVE) {
                int xi = 0;
                for (int n_i = nx; n_i > 1;) {
                    const int half = n_i >> 1;
                    if (pre[xi + half] <= t) xi += half;
                    n_i -= half;
                }
                const int32_t x = A.col[lo[xi] + (t - pre[xi])];
                if (x == v) continue;
                const FdVertex<M> X = info[x];
                const int l1 = lab[xi];
                const bool near = staged ? contains(near_list, d, x) : contains(A.col + r0, d, x);
                if (near) {
                    fd_or(&common[xi], fd_bit<M>(X.lab));
                    // each triangle comes from both of its neighbours of v
                    if (X.lab >= l1) tr.add_new(&tri[l1], l1, L, fd_bit<M>(X.lab));
                }
                M m = fd_less1(X, l1);
                // v itself is x's only other neighbour of its label
                if (near && !(fd_less2(X, l1) & bv)) m &= ~bv;
                pe.add_new(&tab[l1 * L + X.lab], l1 * L + X.lab, L, m);
            }
            wave_sync();   // the common labels are complete
            if (on) {
                const M left = fd_less1(V, W.lab), right = fd_less1(W, lv);
                const M single = left & ~fd_less2(V, W.lab) & right & ~fd_less2(W, lv);
                const M same = left & right & ~(single & common[lane()]);
                if (right & ~inner[W.lab]) fd_or(&inner[W.lab], right);
                if (same & ~diag[W.lab]) fd_or(&diag[W.lab], same);
            }
            wave_sync();   // the next neighbours overwrite the lists
        }
        const int n1 = fd_list((uint64_t)V.m1, list);
        const uint32_t inv = fd_inv(n1);
        T.sync();
        for (int i = T.first; i < n1 * n1; i += T.step) {
            const int q = fd_div(i, inv), l0 = list[q], l2 = list[i - q * n1];
            if (fd_less1(V, l2) & fd_bit<M>(l0))
                pi.add_mask(l0 * L + l2, L, (M)((inner[l2] & ~fd_bit<M>(l0)) | (diag[l2] & fd_bit<M>(l0))));
        }
        T.sync();   // the next vertex clears the masks
    });
    pe.flush(L3, A.pe + (int64_t)lv * L3);
    pi.flush(L3, A.pi + (int64_t)lv * L3);
    tr.flush(L2, A.tr + (int64_t)lv * L2);
}

// A.open from the wedges' supports: a workgroup per leaf label l; its waves take the
// centres in turn, a label of the other leaf per lane.
__global__ __launch_bounds__(512) void k_fd_open(FdArgs A, unsigned long long* __restrict__ open) {
    __shared__ unsigned long long m;
    const int L = A.L, L2 = L * L, l = (int)blockIdx.x;
    if (threadIdx.x == 0) m = 0ull;
    __syncthreads();
    const int a = min(l, lane()), b = max(l, lane());
    for (int c = (int)threadIdx.x / WAVE; c < L; c += (int)blockDim.x / WAVE) {
        uint32_t s = 0;
        if (lane() < L) s = min(A.wc[c * L2 + a * L + b], min(A.wl[a * L2 + c * L + b], A.wl[b * L2 + c * L + a]));
        if (ballot(s > 0 && s >= A.sigma) != 0ull && lane() == 0) atomicOr(&m, 1ull << c);
    }
    __syncthreads();
    if (threadIdx.x == 0) open[l] = m;
}

// Supports: per pattern the smallest of its orbits' domains, 0 below sigma.
// A thread takes one tuple of labels and reports where it is the pattern's
// representative.  *frequent += patterns reported.
__global__ __launch_bounds__(256) void k_fd_supports(FdArgs A, PatBase B, int max_edges,
                                                     const int32_t* __restrict__ path_rank, uint64_t sigma,
                                                     uint64_t* __restrict__ sup,
                                                     unsigned long long* __restrict__ frequent) {
    uint32_t reported = 0;
    const int64_t L = A.L, L2 = L * L, L3 = L2 * L;
    const int64_t N = max_edges >= 3 ? L3 * L : (max_edges == 2 ? L3 : L2);
    auto put = [&](int64_t pid, uint32_t s) {
        if (s >= sigma && s > 0) {
            sup[pid] = s;
            ++reported;
        }
    };
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = i % L, c = i / L % L, b = i / L2 % L, a = i / L3;
        if (max_edges >= 3) {
            const int64_t rev = ((d * L + c) * L + b) * L + a;
            if (i <= rev) {   // path a b c d; its other reading is at least as large
                const uint32_t ends = min(A.pe[i], A.pe[rev]);
                // inner vertices: [label][near end][other inner][far end]
                const uint32_t in1 = A.pi[((b * L + a) * L + c) * L + d], in2 = A.pi[((c * L + d) * L + b) * L + a];
                put(B.path + path_rank[i], min(ends, min(in1, in2)));
            }
            if (b <= c && c <= d) {   // star of centre a, leaves b, c, d
                const uint32_t leaves = min(A.sl[((b * L + a) * L + c) * L + d],
                                            min(A.sl[((c * L + a) * L + b) * L + d], A.sl[((d * L + a) * L + b) * L + c]));
                put(B.star + a * B.t3 + triple_rank(b, c, d, L), min(A.sc[i], leaves));
            }
        }
        if (a != 0) continue;   // three labels b, c, d
        if (max_edges >= 3 && b <= c && c <= d)
            put(B.tri + triple_rank(b, c, d, L),
                min(A.tr[b * L2 + c * L + d], min(A.tr[c * L2 + b * L + d], A.tr[d * L2 + b * L + c])));
        if (max_edges >= 2 && c <= d)   // wedge of centre b
            put(B.wedge + b * B.p2 + pair_rank(c, d, L),
                min(A.wc[b * L2 + c * L + d], min(A.wl[c * L2 + b * L + d], A.wl[d * L2 + b * L + c])));
        if (b == 0 && c <= d) put(B.edge + pair_rank(c, d, L), min(A.edge[c * L + d], A.edge[d * L + c]));
    }
    __shared__ uint32_t total;
    if (threadIdx.x == 0) total = 0u;
    __syncthreads();
    reported = wave_sum_u32(reported);
    if (lane() == 0 && reported) atomicAdd(&total, reported);
    __syncthreads();
    if (threadIdx.x == 0 && total) atomicAdd(frequent, (unsigned long long)total);
}

// Embeddings of two and three edges, for the kernel times' records only: out[0]
// wedges, stars and paths of three edges (a triangle as three of these), out[1]
// triangles, each at the edge of its two smallest ids.  Eight lanes share a vertex's
// edges, the wave those of a longer list (500,000 vertices of 8 neighbours: 773 us with
// a wave per vertex and every common neighbour looked up, 273 so).
constexpr int FD_EMB_LONG = 64;
__global__ __launch_bounds__(256) void k_fd_embeddings(int64_t n, int max_edges, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ col,
                                                       unsigned long long* __restrict__ out) {
    uint64_t sum = 0, triangles = 0;
    // edge (v, col[j]) to an end u of a larger (degree, id), whose list is longer: v's
    // neighbours beyond u and v (those from above on are beyond v), every step-th from
    // the first-th on, are looked up in it
    auto edge = [&](int64_t v, int64_t r0, int64_t r1, int64_t above, int64_t j, int first, int step) {
        const uint64_t d = (uint64_t)(r1 - r0);
        const int32_t u = col[j];
        const int64_t q0 = rp[u];
        const uint64_t du = (uint64_t)(rp[u + 1] - q0);
        if (du < d || (du == d && u < v)) return;
        if (first == 0) sum += (d - 1) * (du - 1);
        for (int64_t i = max64(above, j + 1) + first; i < r1; i += step)
            triangles += contains(col + q0, (int32_t)du, col[i]);
    };
    const int64_t per = (int64_t)(WAVE / 8) * gridDim.x * (blockDim.x / WAVE);
    for (int64_t v0 = (blockIdx.x * (int64_t)(blockDim.x / WAVE) + threadIdx.x / WAVE) * (WAVE / 8); v0 < n; v0 += per) {
        const int64_t v = v0 + lane() / 8;
        const int sub = lane() % 8;
        const int64_t r0 = v < n ? rp[v] : 0, r1 = v < n ? rp[v + 1] : 0;
        const uint64_t d = (uint64_t)(r1 - r0);
        if (sub == 0 && d >= 2) {
            if (max_edges >= 2) sum += d * (d - 1) / 2;
            if (max_edges >= 3) sum += d * (d - 1) * (d - 2) / 6;
        }
        if (max_edges < 3) continue;
        const int64_t above = lower_bound(col, r0, r1, (int32_t)v);
        if (d <= FD_EMB_LONG)
            for (int64_t j = r0 + sub; j < r1; j += 8) edge(v, r0, r1, above, j, 0, 1);
        for (uint64_t more = ballot(sub == 0 && d > FD_EMB_LONG); more; more &= more - 1) {
            const int l = __builtin_ctzll(more);
            const int64_t a = bcast64(r0, l), b = bcast64(r1, l), c = bcast64(above, l);
            for (int64_t j = a; j < b; ++j) edge(v0 + l / 8, a, b, c, j, lane(), WAVE);
        }
    }
    sum = wave_sum_u64(sum);
    triangles = wave_sum_u64(triangles);
    if (lane() == 0 && sum) atomicAdd(&out[0], (unsigned long long)sum);
    if (lane() == 0 && triangles) atomicAdd(&out[1], (unsigned long long)triangles);
}

__global__ void k_fd_label_hist(int64_t n, const int32_t* __restrict__ lab, int L, uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[64];
    if (threadIdx.x < 64) h[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&h[lab[v]], 1u);
    __syncthreads();
    if ((int)threadIdx.x < L && h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

__global__ void k_fd_label_keys(int64_t n, const int32_t* __restrict__ lab, uint64_t* __restrict__ keys) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        keys[v] = ((uint64_t)(uint32_t)lab[v] << 32) | (uint64_t)v;
}

__global__ void k_fd_order(int64_t n, const uint64_t* __restrict__ keys, uint32_t* __restrict__ order) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        order[i] = (uint32_t)keys[i];
}

static unsigned fd_grid(int64_t items) {
    const int64_t b = (items + 255) / 256;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, (int64_t)device_info().n_cu * 16));
}

// Vertices by label and the chunks of one label each: laid out once per graph.
static void build_label_plan(pg_graph* g) {
    LabelPlan& P = g->labels_plan;
    if (P.built) return;
    hipStream_t s = g->stream;
    const int64_t n = g->n;
    const int L = g->n_labels;
    Arena ar;
    SettleOnError settle(s);
    ar.buf.reserve(sizeof(uint64_t) * (size_t)(2 * n) + 256 * 12 * (size_t)(n / 2048 + 2) + (size_t(1) << 20));
    uint32_t* hist = push<uint32_t>(ar, L);
    uint64_t* keys = push<uint64_t>(ar, n);
    uint64_t* tmp = push<uint64_t>(ar, n);
    fill_u32(hist, L, 0, s);
    P.order.reserve(sizeof(uint32_t) * std::max<int64_t>(n, 1));
    if (n > 0) {
        k_fd_label_hist<<<fd_grid(n), 256, 0, s>>>(n, g->labels.as<int32_t>(), L, hist);
        PG_HIP(hipGetLastError());
        k_fd_label_keys<<<fd_grid(n), 256, 0, s>>>(n, g->labels.as<int32_t>(), keys);
        PG_HIP(hipGetLastError());
        radix_sort_u64(keys, tmp, n, 32, 32 + 6, ar, s);   // at most 64 labels; stable, so by id within one
        k_fd_order<<<fd_grid(n), 256, 0, s>>>(n, keys, P.order.as<uint32_t>());
        PG_HIP(hipGetLastError());
    }
    std::vector<uint32_t> h((size_t)L);
    PG_HIP(hipMemcpyAsync(h.data(), hist, sizeof(uint32_t) * L, hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    // about twelve chunks per CU (three or four are resident; 500,000
    // vertices: 2.3 ms a call with four, 1.9 with twelve), of 32 vertices at least (a
    // chunk clears and adds its counters once) and fewer than 2^16 (16-bit
    // counters)
    const int64_t per = std::min<int64_t>(4096, std::max<int64_t>(32, n / (12 * device_info().n_cu)));
    std::vector<int4> chunks;
    int64_t at = 0;
    for (int l = 0; l < L; ++l)
        for (int64_t end = at + h[(size_t)l]; at < end;) {
            const int64_t e = std::min(end, at + per);
            chunks.push_back(make_int4(l, (int)at, (int)e, 0));
            at = e;
        }
    P.n_chunks = (int64_t)chunks.size();
    P.chunks.reserve(sizeof(int4) * std::max<size_t>(chunks.size(), 1));
    if (!chunks.empty())
        PG_HIP(hipMemcpyAsync(P.chunks.p, chunks.data(), sizeof(int4) * chunks.size(), hipMemcpyHostToDevice, s));
    PG_HIP(hipStreamSynchronize(s));
    P.built = true;
}

// Waves per workgroup that the LDS allows beside the chunk's counters, at most 8.
static int fd_waves(int64_t counter_words, int64_t wave_words) {
    const int64_t room = (int64_t(156) << 10) - 4 * counter_words;
    return (int)std::max<int64_t>(0, std::min<int64_t>(8, room / (8 * wave_words)));
}

// Waves from which the counters are held in LDS.  That is up to 32 labels; with 33 a
// single wave is left beside them (50,000 vertices of 8 neighbours: stars 2,985 us, with
// eight waves and counters in device memory 739; paths 1,668 and 1,618).
constexpr int FD_LDS_WAVES = 4;

template <class K>
static void fd_launch(K kernel, FdArgs& A, int waves, int64_t wave_words, int64_t counter_words, int64_t chunks,
                      hipStream_t s) {
    A.waves = waves;
    const size_t lds = (size_t)(8 * wave_words * waves + 4 * counter_words + 16);
    kernel<<<(unsigned)chunks, 64 * waves, lds, s>>>(A);
    PG_HIP(hipGetLastError());
}

template <class M>
static bool fsm_domains(pg_graph* g, int max_edges, uint64_t min_support, uint64_t* supports, size_t* n_frequent) {
    const int64_t n = g->n, L = g->n_labels, L2 = L * L, L3 = L2 * L;
    Arena& ar = g->arena;
    hipStream_t s = g->stream;
    const PatBase B = pat_base(L, max_edges);
    const int64_t np = B.total;
    const int64_t L4 = max_edges >= 3 ? L3 * L : 0;
    // masks, counters and supports have to fit the memory budget
    const uint64_t need = 40 * (uint64_t)n + 4 * (uint64_t)(g->nnz / FD_LONG) + 4 * (uint64_t)(4 * L4 + 4 * L3) + 12 * (uint64_t)L4 + 8 * (uint64_t)np +
                          (uint64_t(1) << 20);
    if (max_edges > 3 || need > g->budget) return false;
    build_label_plan(g);
    const LabelPlan& P = g->labels_plan;
    FdVertex<M>* info = push<FdVertex<M>>(ar, std::max<int64_t>(n, 1));
    const int64_t n_cnt = L2 + 2 * L3 + (max_edges >= 3 ? 4 * L4 + L3 : 0);
    uint32_t* cnt = push<uint32_t>(ar, n_cnt);
    uint64_t* sup = push<uint64_t>(ar, np + FSM_EXTRA + 1);   // then their number, two work counters, long lists
    fill_u32(cnt, n_cnt, 0, s);
    fill_u64(sup, np + FSM_EXTRA + 1, 0, s);
    uint32_t* n_long = reinterpret_cast<uint32_t*>(sup + np + FSM_EXTRA);
    // (the vertices whose lists are at least that long)
    int32_t* long_list = push<int32_t>(ar, (size_t)std::max<int64_t>(1, g->max_deg < FD_LONG ? 0 : g->nnz / FD_LONG));
    FdArgs A{};
    const int64_t* rp = g->rp.as<int64_t>();
    A.col = g->col.as<int32_t>();
    A.info = info;
    A.order = P.order.as<uint32_t>();
    A.chunks = P.chunks.as<int4>();
    A.L = (int)L;
    A.sigma = min_support;
    while ((int64_t(1) << A.lg) < L) ++A.lg;
    A.edge = cnt;
    A.wc = A.edge + L2;
    A.wl = A.wc + L3;
    int32_t* path_rank = nullptr;
    uint64_t* open = nullptr;
    if (max_edges >= 3) {
        A.sc = A.wl + L3;
        A.sl = A.sc + L4;
        A.pe = A.sl + L4;
        A.pi = A.pe + L4;
        A.tr = A.pi + L4;
        open = push<uint64_t>(ar, L);
        A.open = open;
        path_rank = push<int32_t>(ar, L4);
        fsm_path_ranks(L, path_rank, ar, s);
    }
    if (P.n_chunks > 0) {
        {
            ProfScope pw("fsm_masks_work", s, 4.0 * (double)g->nnz * 2 + 52.0 * (double)n);
            ProfScope ps("fsm_masks", s, (double)n);
            k_fd_masks<M><<<fd_grid(8 * n), 256, 0, s>>>(n, rp, A.col, g->labels.as<int32_t>(), info, long_list, n_long);
            PG_HIP(hipGetLastError());
            if (g->max_deg >= FD_LONG) {
                k_fd_long_masks<M><<<(unsigned)(2 * device_info().n_cu), 1024, 0, s>>>(
                    rp, A.col, g->labels.as<int32_t>(), info, long_list, n_long);
                PG_HIP(hipGetLastError());
            }
        }
        // one-step shapes
        const int64_t c1 = (L + 1) / 2 + 2 * ((L2 + 1) / 2);
        const unsigned edge_blocks = (unsigned)std::min<int64_t>(512, (P.n_chunks + 3) / 4);
        if (max_edges == 1) {
            // without the wedges' masks of every neighbour: a million vertices of 4
            // neighbours and 64 labels 1,644 us with them
            ProfScope ps("fsm_stars", s, (double)n);
            k_fd_edges<M><<<edge_blocks, 256, 0, s>>>(A, (int)P.n_chunks);
            PG_HIP(hipGetLastError());
        } else if (max_edges == 2) {
            ProfScope ps("fsm_stars", s, (double)n);
            fd_launch(k_fd_stars<M, false, false, true>, A, 8, fd_words<M>((int)L) + 8, c1, P.n_chunks, s);
        } else {
            const int64_t cs = c1 + 2 * ((L3 + 1) / 2), cq = 2 * ((L3 + 1) / 2) + (L2 + 1) / 2;
            const int64_t ws = fd_words<M>((int)(L2 + L)) + 8;
            const int64_t wq = fd_words<M>((int)(L2 + 3 * L + WAVE)) + 3 * WAVE + 8;
            const int ns = fd_waves(cs, ws), nq = fd_waves(cq, wq);
            // The edges filter the wedges and stars where that may spare much: hubs hold
            // the pass (200,000 vertices with four hubs of 20,000, nothing frequent: 1,012
            // us a call without, 145 with), and where two labels have fewer edges between
            // them than twice the threshold on average, many are infrequent (200,000
            // vertices of 20 neighbours, 29 labels, nothing frequent: 3,015 us without,
            // 563 with).  Elsewhere it only costs: 500,000 vertices of 8 neighbours take
            // 1,539 us without and 1,563 with.
            const bool filter = g->max_deg >= FD_LONG || (double)g->nnz < 2.0 * (double)min_support * (double)L2;
            if (filter) {
                k_fd_edges<M><<<edge_blocks, 256, 0, s>>>(A, (int)P.n_chunks);
                PG_HIP(hipGetLastError());
            }
            {
                ProfScope ps("fsm_stars", s, (double)n);
                if (ns >= FD_LDS_WAVES)
                    fd_launch(filter ? k_fd_stars<M, true, true, true> : k_fd_stars<M, true, false, true>, A, ns, ws, cs,
                              P.n_chunks, s);
                else
                    fd_launch(filter ? k_fd_stars<M, true, true, false> : k_fd_stars<M, true, false, false>, A,
                              fd_waves(0, ws), ws, 0, P.n_chunks, s);
            }
            k_fd_open<<<(unsigned)L, 512, 0, s>>>(A, reinterpret_cast<unsigned long long*>(open));
            PG_HIP(hipGetLastError());
            {
                ProfScope ps("fsm_paths", s, (double)n);
                if (nq >= FD_LDS_WAVES) fd_launch(k_fd_paths<M, true>, A, nq, wq, cq, P.n_chunks, s);
                else fd_launch(k_fd_paths<M, false>, A, fd_waves(0, wq), wq, 0, P.n_chunks, s);
            }
        }
    }
    unsigned long long* work = reinterpret_cast<unsigned long long*>(sup + np);
    const int64_t tuples = max_edges >= 3 ? L4 : L3;
    k_fd_supports<<<std::min(fd_grid(tuples), 1024u), 256, 0, s>>>(A, B, max_edges, path_rank, min_support, sup, work);
    PG_HIP(hipGetLastError());
    if (prof_on() && n > 0) {
        k_fd_embeddings<<<fd_grid(8 * n), 256, 0, s>>>(n, max_edges, rp, A.col, work + 1);
        PG_HIP(hipGetLastError());
    }
    // one copy, straight to the caller's array (14 MB with 40 labels: through an array
    // of its own 5 to 7 ms a call, 4 without)
    PG_HIP(hipMemcpyAsync(supports, sup, sizeof(uint64_t) * (np + FSM_EXTRA), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    const uint64_t* h = supports + np;
    if (prof_on()) {
        // embeddings of up to max_edges edges: a triangle once, not as three paths
        ProfScope ps("fsm_embeddings", s, (double)(g->nnz / 2) + (double)h[1] - 2.0 * (double)h[2]);
    }
    if (n_frequent) *n_frequent = (size_t)h[0];
    return true;
}

bool run_fsm_domains(pg_graph* g, int max_edges, uint64_t min_support, uint64_t* supports, size_t* n_frequent) {
    return g->n_labels <= 32 ? fsm_domains<uint32_t>(g, max_edges, min_support, supports, n_frequent)
                             : fsm_domains<uint64_t>(g, max_edges, min_support, supports, n_frequent);
}

}  // namespace pg
