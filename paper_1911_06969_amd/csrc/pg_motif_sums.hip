// 3- and 4-vertex motif counts from sums over vertices, edges and vertex
// pairs (Pangolin sections 2.2 and 4.2: the counts are those of the
// extend-reduce program, every connected induced subgraph once).
//
// Three vertices: triangles from pg_clique.hip, wedges as the sum over
// vertices of C(d, 2) less three per triangle.
//
// Four vertices: the numbers of (not necessarily induced) subgraphs of each shape determine
// the induced counts, by whole-number combinations:
//   3-stars    sum over vertices of C(d, 3)
//   paths      sum over edges of (d - 1)(d' - 1), less 3 per triangle
//   diamonds   sum over edges of C(t, 2), t = triangles at the edge
//   paws       sum over triangles of the degrees less 2, which is half the
//              sum over edges of t (d + d' - 4)
//   4-cycles   sum over vertex pairs of C(c, 2), c = common neighbours below
//              both, counted at the cycle's first vertex
//   4-cliques  pg_clique.hip
// So what is left to find is t per edge and the pair sum.  Both come from
// one walk over two-step paths a - x - b on the graph renamed by decreasing
// degree, where a is the smaller name (higher degree) of the edge (a, x): b
// adjacent to a is a triangle at (a, x); b > a is one more common neighbour
// x > a of the pair (a, b), and each earlier one closes a 4-cycle whose
// first vertex is a.  Every edge walks the list of its end of lower degree,
// so the walk is short where the graph is skewed: 5.3e8 steps on the
// scale-18 R-MAT graph, where extending every connected 3-set streamed 1.3e11
// candidates.
//
// The common neighbours of (a, .) are counted in LDS by the workgroup that
// holds a: in a table indexed by b where a has many two-step paths (in
// blocks of the vertex range), in a hash table of its own size otherwise.
// An entry's top bit says that b is adjacent to a.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

constexpr int32_t PR_LONG = 256;      // lists of vertices of at least this degree are walked by a whole wave,
constexpr int32_t PR_MID = 24;        // of at least this by a group of lanes, shorter ones by a lane each
constexpr int PR_GROUP = 8;
constexpr int PR_SMALL = 512;         // keys of a one-wave workgroup's hash table (of 1,024 slots, 6 KB)
constexpr int PR_MEDIUM = 4096;       // of a large one's (8,192 slots, 48 KB: three workgroups per CU)
constexpr int PR_MED_THREADS = 256;
constexpr int PR_DIR_THREADS = 1024;
constexpr int PR_DIR_WORDS = 38 << 10;   // LDS words of the indexed table (152 of the 160 KB)
// Vertices of this many steps are shared by several workgroups, each with a
// range of the names and a smaller table (three workgroups per CU).
constexpr int64_t PR_SHARE = 1 << 18;
constexpr int PR_SHARE_THREADS = 512;
constexpr int PR_SHARE_WORDS = 13 << 10;
constexpr int PR_SHARES = 8;          // ranges, of even weight; more where a table would not hold one
constexpr int PR_MAX_SHARES = 16;

// Entry widths of the indexed table: (a, b) have at most deg(b) common
// neighbours, and names follow degrees, so the names fall into runs of entries
// of 32, 16, 8 and 4 bits, of which the top one is the mark.  (On the scale-18
// R-MAT graph the 111,000 names of degree 2 or more take 106 KB, one block;
// with 16 bits for all they take two.)  The first names, which nearly every
// list begins with, have 16 entries each, one per lane modulo 16: lanes that
// add to one address take turns.
constexpr int PR_RUNS = 5;
constexpr int PR_HOT = 256;          // first names
constexpr int PR_COPIES_LOG = 4;
__host__ __device__ constexpr int pr_width(int run) { return run == 0 ? 5 : 6 - run; }   // log2 of an entry's bits
__host__ __device__ constexpr int pr_shift(int run) { return run == 0 ? 5 + PR_COPIES_LOG : 6 - run; }   // of a name's
struct PairRuns {
    int32_t first[PR_RUNS + 1];   // first name of each run; first[PR_RUNS] = n2
};

// A vertex's list, cut after the last vertex of degree 2 or more (n2 names):
// a neighbour of degree 1 is on no triangle or cycle.
struct PairRow {
    int64_t start;
    int32_t len;
    int32_t pad;
};

// A vertex whose walk has something to count: its cut list, its neighbours
// above it (na from `up` on, the first n_long and n_mid of them with long and
// middling lists), its first L1 entry and its hash table's slots.
struct PairItem {
    int64_t start, up, entry;
    int32_t a, len, na, n_long, n_mid;
    uint32_t slots;
};

// The name ranges of shared vertices.  cut[x * n + k]: first place in x's list
// of a name of range k or later.
struct PairShares {
    int32_t n;
    int32_t bound[PR_MAX_SHARES + 1];
    const int32_t* cut;
};

struct PairArgs {
    const int32_t* col;
    const PairRow* row;
    int32_t n2;
    PairRuns runs;
    uint32_t* tri;             // triangles of each L1 entry
    int32_t* done;             // steps of an L1 entry's walk that earlier blocks took
    unsigned long long* out;   // out[2] += 4-cycles
};

// Calls op(u, ok) for the elements of the sorted list at[0, len) below hi, U
// at a time (u[q] counts where ok[q]), with the next U in flight.  G = 1: a
// lane reads neighbouring elements (up to 2 U - 1 past the list: the array is
// padded); else G neighbouring lanes share the list and read neighbouring
// elements.
template <int G, int U, class Op>
__device__ __forceinline__ void pair_walk(const int32_t* at, int32_t len, int32_t hi, Op&& op) {
    if (len <= 0) return;
    constexpr int STEP = U * G;
    int32_t cur[U], nxt[U];
    auto load = [&](int32_t (&u)[U], int32_t j) {
        if constexpr (G == 1) {
            __builtin_memcpy(u, at + j, sizeof(u));
        } else {
#pragma unroll
            for (int q = 0; q < U; ++q) u[q] = at[min(j + q * G, len - 1)];
        }
    };
    int32_t j = G == 1 ? 0 : lane() % G;
    load(cur, j);
    for (; j < len; j += STEP) {
        const bool more = j + STEP < len;
        load(nxt, more ? j + STEP : j);
        bool ok[U];
#pragma unroll
        for (int q = 0; q < U; ++q) ok[q] = j + q * G < len && cur[q] < hi;
        op(cur, ok);
        if (cur[U - 1] >= hi) break;   // the list ascends
#pragma unroll
        for (int q = 0; q < U; ++q) cur[q] = nxt[q];
    }
}

template <int G>
__device__ __forceinline__ uint32_t group_sum(uint32_t v) {
#pragma unroll
    for (int d = G / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, WAVE);
    return v;
}

// A vertex per workgroup, its common-neighbour counts in an open-addressing
// hash table (keys: name << 1 | adjacent to a; 16-bit counts).  The table has
// at least twice as many slots as keys can occur.
template <int NT, int SLOTS>
__global__ __launch_bounds__(NT) void k_pairs_hash(PairArgs A, const PairItem* __restrict__ items, int64_t n_items) {
    __shared__ uint32_t key[SLOTS];
    __shared__ uint32_t cnt[SLOTS / 2];
    constexpr uint32_t EMPTY = ~0u;
    uint64_t cycles = 0;
    for (int64_t i = blockIdx.x; i < n_items; i += gridDim.x) {
        const PairItem I = items[i];
        const int32_t a = uniform(I.a), na = uniform(I.na);
        const uint32_t m = (uint32_t)uniform((int32_t)I.slots);
        const int sh = 32 - (31 - __clz(m));
        auto hash = [&](int32_t b) { return ((uint32_t)b * 0x9E3779B1u) >> sh; };
        for (uint32_t j = threadIdx.x; j < m; j += NT) key[j] = EMPTY;
        for (uint32_t j = threadIdx.x; j < m / 2; j += NT) cnt[j] = 0u;
        __syncthreads();
        for (int32_t j = threadIdx.x; j < I.len; j += NT) {
            const int32_t b = A.col[I.start + j];
            uint32_t h = hash(b);
            while (atomicCAS(&key[h], EMPTY, ((uint32_t)b << 1) | 1u) != EMPTY) h = (h + 1) & (m - 1);
        }
        __syncthreads();
        constexpr int G = NT == WAVE ? 8 : PR_GROUP;   // the one-wave tables' lists are the shorter ones
        for (int32_t j = (int32_t)threadIdx.x / G; j < na; j += NT / G) {
            const PairRow X = A.row[A.col[I.up + j]];
            uint32_t t = 0;
            auto visit = [&](int32_t b) {
                uint32_t h = hash(b);
                while (true) {
                    uint32_t k = key[h];
                    if (k == EMPTY) {
                        if (b <= a) return;   // not adjacent to a, not counted
                        k = atomicCAS(&key[h], EMPTY, (uint32_t)b << 1);
                        if (k == EMPTY) k = (uint32_t)b << 1;
                    }
                    if ((k >> 1) == (uint32_t)b) {
                        t += k & 1u;
                        if (b > a) {
                            const int s = (int)(h & 1u) * 16;
                            cycles += (atomicAdd(&cnt[h >> 1], 1u << s) >> s) & 0xffffu;
                        }
                        return;
                    }
                    h = (h + 1) & (m - 1);
                }
            };
            pair_walk<G, 4>(A.col + X.start, X.len, A.n2, [&](const int32_t (&u)[4], const bool (&ok)[4]) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (ok[q]) visit(u[q]);
            });
            t = group_sum<G>(t);
            if (lane() % G == 0) A.tri[I.entry + j] = t;
        }
        __syncthreads();   // the next vertex clears the table
    }
    cycles = wave_sum_u64(cycles);
    if (lane() == 0 && cycles) atomicAdd(&A.out[2], (unsigned long long)cycles);
}

// A vertex per workgroup, its common-neighbour counts in a table indexed by
// b, in blocks of the names where one table does not hold them all (a list's
// walk goes on where the block before stopped).  SHARED: a range of the names
// per workgroup, from the lists' stored cuts; a hub of 15,800 neighbours and
// 2.5e6 steps takes one workgroup 1.4 ms (it waits on the loads of 16 waves).
// Long lists are walked by whole waves, middling ones by PR_GROUP lanes (both
// coalesced), the others by a lane each: names follow degrees, so the lists
// of neighbouring lanes are of similar lengths.
template <bool SHARED>
__global__ __launch_bounds__(SHARED ? PR_SHARE_THREADS : PR_DIR_THREADS)
    void k_pairs_indexed(PairArgs A, PairShares H, const PairItem* __restrict__ items, int64_t n_items,
                         unsigned long long* __restrict__ next) {
    extern __shared__ __align__(16) uint32_t table[];
    __shared__ int64_t s_item;
    constexpr int NT = SHARED ? PR_SHARE_THREADS : PR_DIR_THREADS;
    constexpr int64_t TABLE_BITS = 32ll * (SHARED ? PR_SHARE_WORDS : PR_DIR_WORDS);
    uint64_t cycles = 0;
    while (true) {
        if (threadIdx.x == 0) s_item = (int64_t)atomicAdd(next, 1ull);
        __syncthreads();
        const int64_t it = uniform64(s_item);
        if (it >= n_items) break;
        const int range = SHARED ? (int)(it % H.n) : 0;
        const PairItem I = items[SHARED ? it / H.n : it];
        const int32_t a = uniform(I.a), na = uniform(I.na);
        const int32_t n_long = uniform(I.n_long), n_mid = uniform(I.n_mid);
        const int32_t end = SHARED ? H.bound[range + 1] : A.n2;
        for (int32_t lo = SHARED ? H.bound[range] : 0; lo < end;) {
            // the block's names [lo, hi): the runs from lo on while they fit;
            // run r's entry of b is at bit off[r] + (b << shift)
            int32_t off[PR_RUNS];
            int32_t hi = lo;
            int64_t bits = 0;
#pragma unroll
            for (int r = 0; r < PR_RUNS; ++r) {
                const int32_t f = max(A.runs.first[r], lo), e = min(A.runs.first[r + 1], end);
                bits = (bits + 31) & ~31ll;
                off[r] = (int32_t)(bits - ((int64_t)f << pr_shift(r)));   // modulo 2^32
                if (hi == f && f < e) {
                    hi = f + (int32_t)min64(e - f, max64(TABLE_BITS - bits, 0) >> pr_shift(r));
                    bits += (int64_t)(hi - f) << pr_shift(r);
                }
            }
            // bit of b's entry (of the lane's, for a first name), and log2 of
            // its width
            const int copy = lane() & ((1 << PR_COPIES_LOG) - 1);
            auto place = [&](int32_t b, int& wd) {
                uint32_t p = (uint32_t)off[0] + ((uint32_t)b << pr_shift(0)) + ((uint32_t)copy << 5);
                wd = pr_width(0);
#pragma unroll
                for (int r = 1; r < PR_RUNS; ++r)
                    if (b >= A.runs.first[r]) {
                        wd = pr_width(r);
                        p = (uint32_t)off[r] + ((uint32_t)b << pr_shift(r));
                    }
                return p;
            };
            const int32_t hot = A.runs.first[1];
            const int words = (int)((bits + 127) / 128);   // of four
            for (int j = threadIdx.x; j < words; j += NT)
                reinterpret_cast<uint4*>(table)[j] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            for (int32_t j = threadIdx.x; j < I.len; j += NT) {
                const int32_t b = A.col[I.start + j];
                if (b >= lo && b < hi) {
                    int wd;
                    const uint32_t p = place(b, wd), bit = 1u << ((p & 31) + (1 << wd) - 1);
                    const uint32_t w = b < hot ? (p >> 5) - copy : p >> 5;
                    const int copies = b < hot ? 1 << PR_COPIES_LOG : 1;
                    for (int c = 0; c < copies; ++c) atomicOr(&table[w + c], bit);
                }
            }
            __syncthreads();
            uint32_t t = 0;
            int32_t steps = 0;
            // neighbours [j0, j1) in a's order, G lanes each; the next one's
            // row is loaded during the walk
            auto walk = [&](auto gc, auto uc, int32_t j0, int32_t j1) {
                constexpr int G = decltype(gc)::value, U = decltype(uc)::value;
                // U counts are taken together; idle lanes add nothing to an
                // entry of their own
                auto visit = [&](const int32_t (&u)[U], const bool (&ok)[U]) {
                    uint32_t o[U];
                    uint32_t pos[U];
                    int wd[U];
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        pos[q] = place(u[q], wd[q]);
                        const uint32_t add = ok[q] && u[q] > a ? 1u : 0u;
                        o[q] = atomicAdd(&table[ok[q] ? pos[q] >> 5 : lane()], add << (pos[q] & 31));
                    }
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        const int wid = 1 << wd[q];
                        const uint32_t c = o[q] >> (pos[q] & 31);
                        t += ok[q] ? (c >> (wid - 1)) & 1u : 0u;
                        cycles += ok[q] && u[q] > a && u[q] >= hot ? c & ((1u << (wid - 1)) - 1u) : 0u;
                        steps += ok[q];
                    }
                };
                int32_t j = j0 + (int32_t)threadIdx.x / G;
                PairRow nx{0, 0, 0};   // the part of the next list to walk
                int32_t nd = 0;        // places before it
                auto fetch = [&](int32_t i) {
                    const int32_t x = A.col[I.up + i];
                    nx = A.row[x];
                    if constexpr (SHARED) {
                        const int32_t* cut = H.cut + (int64_t)x * H.n + range;
                        nd = cut[0];
                        if (range + 1 < H.n) nx.len = cut[1];
                    } else {
                        nd = lo > 0 ? A.done[I.entry + i] : 0;
                    }
                    nx.start += nd;
                    nx.len -= nd;
                };
                if (j < j1) fetch(j);
                for (; j < j1; j += NT / G) {
                    const PairRow X = nx;
                    const int32_t d = nd;
                    if (j + NT / G < j1) fetch(j + NT / G);
                    t = 0;
                    steps = 0;
                    pair_walk<G, U>(A.col + X.start, X.len, hi, visit);
                    t = group_sum<G>(t);
                    if (!SHARED && hi < end) steps = (int32_t)group_sum<G>((uint32_t)steps);
                    if (lane() % G == 0) {
                        if (t) atomicAdd(&A.tri[I.entry + j], t);
                        if (!SHARED && hi < end) A.done[I.entry + j] = d + steps;
                    }
                }
            };
            // a walk step takes U elements per lane whether the list has them
            // or not, so the lanes per list follow the lists' lengths
            using std::integral_constant;
            constexpr integral_constant<int, 4> four{};
            if constexpr (SHARED) {
                walk(integral_constant<int, PR_GROUP>{}, four, 0, n_long);
                walk(integral_constant<int, 1>{}, four, n_long, na);
            } else {
                walk(integral_constant<int, WAVE>{}, four, 0, n_long);
                walk(integral_constant<int, PR_GROUP>{}, four, n_long, n_mid);
                walk(integral_constant<int, 1>{}, four, n_mid, na);
            }
            __syncthreads();
            // the first names' entries together
            for (int32_t b = lo + (int32_t)threadIdx.x; b < min(hi, hot); b += NT) {
                uint64_t c = 0;
                for (int i = 0; i < 1 << PR_COPIES_LOG; ++i)
                    c += table[(((uint32_t)off[0] + ((uint32_t)b << pr_shift(0))) >> 5) + i] & 0x7fffffffu;
                cycles += c * (c - 1) / 2;
            }
            __syncthreads();   // the next block clears the table; `done` is read by the lanes that wrote it
            lo = hi;
        }
    }
    cycles = wave_sum_u64(cycles);
    if (lane() == 0 && cycles) atomicAdd(&A.out[2], (unsigned long long)cycles);
}

// C(d, 3) modulo 2^64
__device__ __forceinline__ uint64_t choose3(uint64_t d) {
    if (d < 3) return 0;
    uint64_t f[3] = {d, d - 1, d - 2};
    if (f[0] & 1) f[1] >>= 1; else f[0] >>= 1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // d and d - 1 were halved where even, which keeps a factor of 3
        if (f[i] % 3 == 0) {
            f[i] /= 3;
            break;
        }
    }
    return f[0] * f[1] * f[2];
}

// Sums over vertices and L1 entries: out[0] stars, out[1] paths, out[3] and
// out[4] the low and high 32-bit halves of t (d + d' - 4), out[5] diamonds,
// out[6] t.
__global__ __launch_bounds__(256) void k_pair_sums(int64_t n, int64_t m, const int64_t* __restrict__ rp,
                                                   const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                   const uint32_t* __restrict__ tri,
                                                   unsigned long long* __restrict__ out) {
    uint64_t star = 0, path = 0, lo = 0, hi = 0, dia = 0, ts = 0;
    const int64_t first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = first; v < n; v += step) star += choose3((uint64_t)(rp[v + 1] - rp[v]));
    for (int64_t e = first; e < m; e += step) {
        const int32_t a = src[e], x = dst[e];
        const uint64_t da = (uint64_t)(rp[a + 1] - rp[a]), dx = (uint64_t)(rp[x + 1] - rp[x]);
        const uint64_t t = tri[e];
        path += (da - 1) * (dx - 1);
        if (t) {   // both degrees are at least 2 then
            const uint64_t p = t * (da + dx - 4);
            lo += p & 0xffffffffu;
            hi += p >> 32;
            dia += t * (t - 1) / 2;
            ts += t;
        }
    }
    // one atomic per workgroup and sum (one per wave of 2,048 workgroups took
    // 390 us of a 400 us pass: they queue on one cache line)
    __shared__ uint64_t part[256 / WAVE][6];
    const uint64_t v[6] = {star, path, lo, hi, dia, ts};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const uint64_t s = wave_sum_u64(v[i]);
        if (lane() == 0) part[threadIdx.x / WAVE][i] = s;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        uint64_t s = 0;
        for (int w = 0; w < 256 / WAVE; ++w) s += part[w][threadIdx.x];
        if (s) atomicAdd(&out[threadIdx.x < 2 ? threadIdx.x : threadIdx.x + 1], (unsigned long long)s);
    }
}

// Sum over vertices of C(d, 2).
__global__ __launch_bounds__(256) void k_wedges(int64_t n, const int64_t* __restrict__ rp,
                                                unsigned long long* __restrict__ out) {
    uint64_t sum = 0;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t d = (uint64_t)(rp[v + 1] - rp[v]);
        sum += d * (d - 1) / 2;
    }
    __shared__ uint64_t part[256 / WAVE];
    sum = wave_sum_u64(sum);
    if (lane() == 0) part[threadIdx.x / WAVE] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / WAVE; ++w) sum += part[w];
        if (sum) atomicAdd(out, (unsigned long long)sum);
    }
}

// Wedges (with triangles) and triangles of a small graph from its CSR alone, without
// the DAG and its plan, whose launches and allocations are most of a first call: 16
// lanes per entry (v, u), u > v, take the shorter list's vertices past u and search the
// longer.  out[0] += sum of C(d, 2), out[1] += triangles.  First and later calls, by
// the plan and so: 40 vertices 318, 59 and 38, 31 us; 20,000 of 10 neighbours 398, 69
// and 61, 56.  A hub's entries wait for its lists: R-MAT scale 14 (228,000 entries,
// degrees up to 2,400) 72 us a later call by the plan, 126 so.
constexpr int64_t M3_SMALL = 1 << 18;   // entries
constexpr int64_t M3_DEG = 1024;        // largest degree
__global__ __launch_bounds__(256) void k_motif3_small(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                      const int32_t* __restrict__ col,
                                                      unsigned long long* __restrict__ out) {
    constexpr int G = 16;
    uint64_t wedges = 0, triangles = 0;
    const int64_t first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = first; v < n; v += step) {
        const uint64_t d = (uint64_t)(rp[v + 1] - rp[v]);
        wedges += d * (d - 1) / 2;
    }
    for (int64_t j = first / G; j < nnz; j += step / G) {
        int64_t lo = 0, hi = n - 1;   // the first row that ends past j
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (rp[mid + 1] <= j) lo = mid + 1; else hi = mid;
        }
        const int32_t u = col[j];
        if (u < lo) continue;
        int64_t a = j + 1, b = rp[u];   // v's neighbours past u, u's list
        int32_t na = (int32_t)(rp[lo + 1] - a), nb = (int32_t)(rp[u + 1] - b);
        if (na > nb) {
            const int64_t t = a;
            a = b;
            b = t;
            const int32_t m = na;
            na = nb;
            nb = m;
        }
        for (int32_t i = lane() % G; i < na; i += G) {
            const int32_t x = col[a + i];
            triangles += x > u && contains(col + b, nb, x);
        }
    }
    __shared__ uint64_t part[256 / WAVE][2];
    wedges = wave_sum_u64(wedges);
    triangles = wave_sum_u64(triangles);
    if (lane() == 0) {
        part[threadIdx.x / WAVE][0] = wedges;
        part[threadIdx.x / WAVE][1] = triangles;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint64_t s = 0;
        for (int w = 0; w < 256 / WAVE; ++w) s += part[w][threadIdx.x];
        if (s) atomicAdd(&out[threadIdx.x], (unsigned long long)s);
    }
}

// ------------------------------------------------------------------ plan
//
// The cut lists and the vertices by the kind of table their walk takes depend
// on the graph only; they are kept with the renamed graph.

// counts[i] = names of degree bound[i] or more
struct PairBounds {
    int64_t deg[6];
};
constexpr PairBounds PR_BOUNDS = {{2, 8, 128, 32768, PR_MID, PR_LONG}};   // 8, 128, 32768: the runs

__global__ void k_pair_bounds(int64_t n, const int64_t* __restrict__ rp, PairBounds B, uint64_t* __restrict__ counts) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = rp[v + 1] - rp[v], d1 = v + 1 < n ? rp[v + 2] - rp[v + 1] : 0;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            if (d >= B.deg[i] && d1 < B.deg[i]) counts[i] = (uint64_t)(v + 1);
    }
}

__global__ void k_pair_cut(int64_t n2, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                           PairRow* __restrict__ row) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n2; v += (int64_t)gridDim.x * blockDim.x)
        row[v] = PairRow{rp[v], (int32_t)(lower_bound(col, rp[v], rp[v + 1], (int32_t)n2) - rp[v]), 0};
}

// per L1 entry (a, x): steps of its walk, and those to names above a
__global__ void k_pair_lens(int64_t m, int64_t n2, const int32_t* __restrict__ dst, const int32_t* __restrict__ rev,
                            const PairRow* __restrict__ row, uint32_t* __restrict__ all,
                            uint32_t* __restrict__ above) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = dst[e];
        const int32_t d = x < n2 ? row[x].len : 0;
        all[e] = (uint32_t)d;
        above[e] = (uint32_t)max(d - rev[e], 0);
    }
}

enum { PC_NONE = 0, PC_SMALL, PC_MEDIUM, PC_INDEXED, PC_SHARED };

__global__ void k_pair_class(int64_t n2, const int64_t* __restrict__ rp, const int64_t* __restrict__ seg,
                             const PairRow* __restrict__ row, const uint64_t* __restrict__ all,
                             const uint64_t* __restrict__ above, uint64_t share, uint8_t* __restrict__ cls,
                             uint32_t* __restrict__ slots) {
    for (int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; a < n2; a += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s0 = seg[a], s1 = seg[a + 1];
        const int64_t na = row[a].len - ((rp[a + 1] - rp[a]) - (s1 - s0));   // neighbours in (a, n2)
        uint8_t c = PC_NONE;
        uint32_t sl = 0;
        // a list holding a alone takes part in nothing
        if (na > 0 && (int64_t)(all[s1] - all[s0]) > na) {
            const uint64_t keys = (above[s1] - above[s0]) + (uint64_t)row[a].len;
            if (keys <= (uint64_t)PR_MEDIUM) {
                c = keys <= (uint64_t)PR_SMALL ? PC_SMALL : PC_MEDIUM;
                sl = 64;
                while (sl < 2 * (uint32_t)keys) sl <<= 1;
            } else {
                c = all[s1] - all[s0] >= share ? PC_SHARED : PC_INDEXED;
            }
        }
        cls[a] = c;
        slots[a] = sl;
    }
}

__global__ void k_pair_flags(int64_t n2, const uint8_t* __restrict__ cls, int c, uint32_t* __restrict__ flag) {
    for (int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; a < n2; a += (int64_t)gridDim.x * blockDim.x)
        flag[a] = cls[a] == c ? 1u : 0u;
}

__global__ void k_pair_items(int64_t n2, int32_t x_long, int32_t x_mid, const uint32_t* __restrict__ flag,
                             const uint64_t* __restrict__ pos, const uint32_t* __restrict__ slots,
                             const int64_t* __restrict__ rp, const int64_t* __restrict__ seg,
                             const int32_t* __restrict__ col, const PairRow* __restrict__ row,
                             PairItem* __restrict__ items) {
    for (int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; a < n2; a += (int64_t)gridDim.x * blockDim.x)
        if (flag[a]) {
            PairItem I;
            I.start = rp[a];
            I.up = rp[a + 1] - (seg[a + 1] - seg[a]);
            I.entry = seg[a];
            I.a = (int32_t)a;
            I.len = row[a].len;
            const int64_t end = I.start + I.len;
            I.na = (int32_t)(end - I.up);
            // names ascend in the list and degrees descend: longer lists first
            I.n_long = (int32_t)(lower_bound(col, I.up, end, x_long) - I.up);
            I.n_mid = (int32_t)(lower_bound(col, I.up, end, x_mid) - I.up);
            I.slots = slots[a];
            items[pos[a]] = I;
        }
}

// range bounds of even weight: bound[k] = first name with k / PR_SHARES of the
// entries before it
__global__ void k_pair_shares(int64_t n2, const int64_t* __restrict__ rp, int64_t* __restrict__ bound) {
    const int k = threadIdx.x;
    if (k > PR_SHARES) return;
    const int64_t want = rp[n2] * k / PR_SHARES;
    int64_t lo = 0, hi = n2;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rp[mid] < want) lo = mid + 1; else hi = mid;
    }
    bound[k] = k == PR_SHARES ? n2 : lo;
}

__global__ void k_pair_cuts(int64_t n2, PairShares H, const int32_t* __restrict__ col, const PairRow* __restrict__ row,
                            int32_t* __restrict__ cut) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n2 * H.n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t x = i / H.n;
        const int k = (int)(i % H.n);
        const PairRow X = row[x];
        cut[i] = (int32_t)lower_bound(col + X.start, 0, X.len, H.bound[k]);
    }
}

static unsigned pr_grid(int64_t items) {
    const int64_t b = (items + 255) / 256;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, (int64_t)device_info().n_cu * 16));
}

static PairShares shares_of(const PairPlan& P) {
    PairShares H{};
    H.n = P.shares;
    for (int k = 0; k <= P.shares; ++k) H.bound[k] = P.bound[k];
    H.cut = P.cut.as<int32_t>();
    return H;
}

// Table bits of the names [lo, hi).
static int64_t pair_bits(const PairPlan& P, int64_t lo, int64_t hi) {
    int64_t bits = 0;
    for (int r = 0; r < PR_RUNS; ++r) {
        const int64_t f = std::max<int64_t>(P.run[r], lo), e = std::min<int64_t>(P.run[r + 1], hi);
        if (f < e) bits = ((bits + 31) & ~int64_t(31)) + ((e - f) << pr_shift(r));
    }
    return bits;
}

// The name ranges of shared vertices: of even weight, cut further where a
// table would not hold one; none when that takes more than PR_MAX_SHARES.
static void plan_shares(PairPlan& P, const MotifView& V, Arena& ar, hipStream_t s) {
    int64_t even[PR_SHARES + 1];
    int64_t* d = push<int64_t>(ar, PR_SHARES + 1);
    k_pair_shares<<<1, WAVE, 0, s>>>(P.n2, V.rp, d);
    PG_HIP(hipGetLastError());
    PG_HIP(hipMemcpyAsync(even, d, sizeof(even), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    P.shares = 0;
    P.bound[0] = 0;
    for (int k = 1; k <= PR_SHARES;) {
        const int64_t lo = P.bound[P.shares];
        int64_t hi = even[k];
        if (hi <= lo) {
            ++k;
            continue;
        }
        if (P.shares == PR_MAX_SHARES) {
            P.shares = 0;
            return;
        }
        if (pair_bits(P, lo, hi) > 32ll * PR_SHARE_WORDS) {
            int64_t a = lo + 1, b = hi;   // the largest end whose names fit
            while (a < b) {
                const int64_t mid = (a + b + 1) / 2;
                if (pair_bits(P, lo, mid) <= 32ll * PR_SHARE_WORDS) a = mid; else b = mid - 1;
            }
            hi = a;
        } else {
            ++k;
        }
        P.bound[++P.shares] = (int32_t)hi;
    }
}

static void build_pair_plan(pg_graph* g, const MotifView& V) {
    PairPlan& P = g->mg.pairs;
    if (P.built) return;
    hipStream_t s = g->stream;
    const int64_t n = V.n, m = V.ml1->n_edges;
    const int64_t* seg = V.ml1->seg.as<int64_t>();
    Arena ar;
    SettleOnError settle(s);
    ar.buf.reserve((size_t)(26 * m + 32 * n) + (size_t)(m + n) / 64 + (size_t(1) << 20));
    uint64_t* bounds = push<uint64_t>(ar, 6);
    fill_u64(bounds, 6, 0, s);
    k_pair_bounds<<<pr_grid(n), 256, 0, s>>>(n, V.rp, PR_BOUNDS, bounds);
    PG_HIP(hipGetLastError());
    uint64_t hb[6];
    PG_HIP(hipMemcpyAsync(hb, bounds, sizeof(hb), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    const int64_t n2 = (int64_t)hb[0];
    P.n2 = n2;
    const int64_t hot = std::min<int64_t>(n2, PR_HOT);
    P.run[0] = 0;
    P.run[1] = (int32_t)hot;
    for (int r = 2; r < PR_RUNS; ++r) P.run[r] = (int32_t)std::max<int64_t>(hot, (int64_t)hb[5 - r]);
    P.run[PR_RUNS] = (int32_t)n2;
    for (int64_t& c : P.count) c = 0;
    P.steps = 0;
    P.row.reserve(sizeof(PairRow) * std::max<int64_t>(n2, 1));
    PairRow* row = P.row.as<PairRow>();
    if (n2 > 0) {
        k_pair_cut<<<pr_grid(n2), 256, 0, s>>>(n2, V.rp, V.col, row);
        PG_HIP(hipGetLastError());
        plan_shares(P, V, ar, s);
        if (P.shares > 0) {
            P.cut.reserve(sizeof(int32_t) * (size_t)(n2 * P.shares));
            k_pair_cuts<<<pr_grid(n2 * P.shares), 256, 0, s>>>(n2, shares_of(P), V.col, row, P.cut.as<int32_t>());
            PG_HIP(hipGetLastError());
        }
        uint32_t* all = push<uint32_t>(ar, m);
        uint32_t* above = push<uint32_t>(ar, m);
        uint64_t* all_pre = push<uint64_t>(ar, m + 1);
        uint64_t* above_pre = push<uint64_t>(ar, m + 1);
        k_pair_lens<<<pr_grid(m), 256, 0, s>>>(m, n2, V.ml1->dst.as<int32_t>(), V.ml1->rev.as<int32_t>(), row,
                                               all, above);
        PG_HIP(hipGetLastError());
        scan_u32(all, m, all_pre, ar, s);
        scan_u32(above, m, above_pre, ar, s);
        uint8_t* cls = push<uint8_t>(ar, n2);
        uint32_t* slots = push<uint32_t>(ar, n2);
        uint32_t* flag = push<uint32_t>(ar, n2);
        uint64_t* pos = push<uint64_t>(ar, n2 + 1);
        k_pair_class<<<pr_grid(n2), 256, 0, s>>>(n2, V.rp, seg, row, all_pre, above_pre,
                                                 P.shares > 0 ? (uint64_t)PR_SHARE : UINT64_MAX, cls, slots);
        PG_HIP(hipGetLastError());
        for (int c = PC_SMALL; c <= PC_SHARED; ++c) {
            k_pair_flags<<<pr_grid(n2), 256, 0, s>>>(n2, cls, c, flag);
            PG_HIP(hipGetLastError());
            scan_u32(flag, n2, pos, ar, s);
            const int64_t count = (int64_t)read_u64(pos + n2, s);
            P.count[c - 1] = count;
            P.items[c - 1].reserve(sizeof(PairItem) * std::max<int64_t>(count, 1));
            if (count == 0) continue;
            k_pair_items<<<pr_grid(n2), 256, 0, s>>>(n2, (int32_t)hb[5], (int32_t)hb[4], flag, pos, slots, V.rp, seg,
                                                     V.col, row, P.items[c - 1].as<PairItem>());
            PG_HIP(hipGetLastError());
        }
        P.steps = (double)read_u64(all_pre + m, s);
    }
    PG_HIP(hipStreamSynchronize(s));
    P.built = true;
}

// ------------------------------------------------------------------ host

void count_motifs3(pg_graph* g, uint64_t* counts) {
    hipStream_t s = g->stream;
    Arena& ar = g->arena;
    uint64_t* wedges = push<uint64_t>(ar, 2);
    fill_u64(wedges, 2, 0, s);
    if (g->nnz <= M3_SMALL && g->max_deg <= M3_DEG) {
        ProfScope ps("motif_small", s, (double)g->nnz);
        const int64_t blocks = (std::max<int64_t>(g->n, 16 * g->nnz) + 255) / 256;
        k_motif3_small<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>(blocks, 8 * device_info().n_cu)), 256, 0, s>>>(
            g->n, g->nnz, g->rp.as<int64_t>(), g->col.as<int32_t>(), reinterpret_cast<unsigned long long*>(wedges));
        PG_HIP(hipGetLastError());
        uint64_t h[2];
        PG_HIP(hipMemcpyAsync(h, wedges, sizeof(h), hipMemcpyDeviceToHost, s));
        PG_HIP(hipStreamSynchronize(s));
        counts[0] = h[0] - 3 * h[1];
        counts[1] = h[1];
        return;
    }
    k_wedges<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>((g->n + 1023) / 1024, device_info().n_cu)), 256, 0, s>>>(
        g->n, g->rp.as<int64_t>(), reinterpret_cast<unsigned long long*>(wedges));
    PG_HIP(hipGetLastError());
    const uint64_t triangles = count_cliques(g, 3, true);
    counts[0] = read_u64(wedges, s) - 3 * triangles;
    counts[1] = triangles;
}

void count_motifs4(pg_graph* g, uint64_t* counts) {
    if (count_motifs4_small(g, counts)) return;
    const MotifView V = motif_view(g, true);
    build_motif_l1(g, V);
    const int64_t m = V.ml1->n_edges;
    for (int i = 0; i < 6; ++i) counts[i] = 0;
    if (m == 0) return;
    build_pair_plan(g, V);
    const PairPlan& P = g->mg.pairs;
    hipStream_t s = g->stream;
    Arena& ar = g->arena;
    size_t mk = ar.mark();
    const uint64_t k4 = count_cliques(g, 4, true);
    ar.reset(mk);
    uint64_t* out = push<uint64_t>(ar, 8);
    uint32_t* tri = push<uint32_t>(ar, m);
    fill_u64(out, 8, 0, s);
    fill_u32(tri, m, 0, s);
    PairArgs A{};
    A.col = V.col;
    A.row = P.row.as<PairRow>();
    A.n2 = (int32_t)P.n2;
    A.tri = tri;
    A.out = reinterpret_cast<unsigned long long*>(out);
    for (int r = 0; r <= PR_RUNS; ++r) A.runs.first[r] = P.run[r];
    // one block of names unless their table exceeds the LDS
    const int64_t bits = pair_bits(P, 0, P.n2);
    A.done = bits > 32ll * PR_DIR_WORDS ? push<int32_t>(ar, m) : nullptr;
    const auto lds = [](int64_t b, int words) {
        return (size_t)std::max<int64_t>(std::min<int64_t>(b, 32ll * words) / 128 + 1, WAVE / 4) * 16;
    };
    unsigned long long* next = A.out + 7;
    {
        // 4 B per step; per list its vertex, row start, cut length and result
        ProfScope pw("motif_pairs_work", s, 4.0 * P.steps + 20.0 * (double)m);
        ProfScope ps("motif_pairs", s, P.steps);
        const PairShares H = shares_of(P);
        if (P.count[3] > 0) {
            int64_t most = 0;
            for (int k = 0; k < H.n; ++k) most = std::max(most, pair_bits(P, H.bound[k], H.bound[k + 1]));
            fill_u64(reinterpret_cast<uint64_t*>(next), 1, 0, s);
            const int64_t n = P.count[3] * H.n;
            k_pairs_indexed<true><<<(unsigned)std::min<int64_t>(n, 4 * device_info().n_cu), PR_SHARE_THREADS,
                                    lds(most, PR_SHARE_WORDS), s>>>(A, H, P.items[3].as<PairItem>(), n, next);
            PG_HIP(hipGetLastError());
        }
        if (P.count[2] > 0) {
            fill_u64(reinterpret_cast<uint64_t*>(next), 1, 0, s);
            k_pairs_indexed<false><<<(unsigned)std::min<int64_t>(P.count[2], 2 * device_info().n_cu), PR_DIR_THREADS,
                                     lds(bits, PR_DIR_WORDS), s>>>(A, H, P.items[2].as<PairItem>(), P.count[2], next);
            PG_HIP(hipGetLastError());
        }
        if (P.count[1] > 0) {
            k_pairs_hash<PR_MED_THREADS, 2 * PR_MEDIUM>
                <<<(unsigned)std::min<int64_t>(P.count[1], 12 * device_info().n_cu), PR_MED_THREADS, 0, s>>>(
                    A, P.items[1].as<PairItem>(), P.count[1]);
            PG_HIP(hipGetLastError());
        }
        if (P.count[0] > 0) {
            k_pairs_hash<WAVE, 2 * PR_SMALL>
                <<<(unsigned)std::min<int64_t>(P.count[0], 64 * device_info().n_cu), WAVE, 0, s>>>(
                    A, P.items[0].as<PairItem>(), P.count[0]);
            PG_HIP(hipGetLastError());
        }
    }
    {
        ProfScope ps("motif_sums", s, (double)m);
        k_pair_sums<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>((std::max(V.n, m) + 1023) / 1024, device_info().n_cu)), 256, 0,
                      s>>>(V.n, m, V.rp, V.ml1->src.as<int32_t>(), V.ml1->dst.as<int32_t>(), tri, A.out);
        PG_HIP(hipGetLastError());
    }
    uint64_t h[8];
    PG_HIP(hipMemcpyAsync(h, out, sizeof(h), hipMemcpyDeviceToHost, s));
    PG_HIP(hipStreamSynchronize(s));
    ar.reset(mk);
    const uint64_t paw = (uint64_t)((((unsigned __int128)h[4] << 32) + h[3]) / 2);
    counts[5] = k4;
    counts[4] = h[5] - 6 * k4;
    counts[3] = paw - 4 * counts[4] - 12 * k4;
    counts[2] = h[2] - counts[4] - 3 * k4;
    counts[1] = h[0] - counts[3] - 2 * counts[4] - 4 * k4;
    counts[0] = h[1] - h[6] - 2 * counts[3] - 4 * counts[2] - 6 * counts[4] - 12 * k4;   // h[6]: 3 per triangle
}

}  // namespace pg
