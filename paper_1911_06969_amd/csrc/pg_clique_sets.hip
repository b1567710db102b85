// Last levels of the clique counts: triangles inside sets of siblings.
//
// The k-cliques below an entry of level k - 4 (k = 4: a root, k = 5: an edge of
// the DAG) are the triangles among the vertices that extend it, which the mask
// rows hold as a set S of positions of the root's out-list.  With A the matrix
// of the rows, cut to S, they are the sum of (A A^T) over A's own positions:
// a product on the matrix cores instead of a walk over the edges in S.
//
// A set within one word of the rows (most of the small ones) is counted from
// that word of its rows, a row per lane.  Other sets are first packed: member x
// gets the bits of its row at the members' places, so that a set of n members
// costs n / 64 words a row whatever the out-degree of the root.  Packed rows lie in
// LDS, cut below the diagonal and with an odd number of dwords from row to row
// (a column of rows is then read without bank conflicts).
//
// Measured on R-MAT graphs, against storing every entry of the level above and
// adding popcounts of row pairs: 4-cliques of scale 21, edge factor 13 (607
// million triangles) 3.29 -> 1.06 ms; 5-cliques of a million vertices, edge
// factor 10 (134 million triangles, 3.3 billion cliques) 27.5 -> 4.7 ms.  The
// 5-clique kernel of the wide roots is bound by issue: vector and scalar
// instructions each take 75 % of its cycles (per entry, some 280 of either).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pg_clique.h"
#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

namespace {

constexpr int ST_THREADS = 256;
constexpr int ST_WAVES = ST_THREADS / WAVE;
// members of a packed set at most: with 192 seven workgroups of narrow roots fit
// a CU's LDS (six would with 256); larger sets, found in wider roots only and dense
// there, are counted from the whole rows
constexpr int ST_N = 192;
constexpr int ST_PART = 16;              // entries a wave takes at once

// Rows of 64 nw positions: group q of 64 rows holds the dwords 2q .. 2nw - 1.
__host__ __device__ constexpr int packed_stride(int q, int nw) { return 2 * (nw - q) + 1; }
__host__ __device__ constexpr int packed_base(int q, int nw) { return 64 * q * (2 * nw - q + 2); }
__host__ __device__ constexpr int packed_dwords(int nw) { return packed_base(nw, nw); }

struct PackedRows {
    const uint32_t* B;
    int nw;
    // dword c >= 2q of row 64q + i
    __device__ __forceinline__ uint32_t get(int q, int i, int c) const {
        return B[packed_base(q, nw) + i * packed_stride(q, nw) + c - 2 * q];
    }
};

// A root's block of rows: packed in LDS, or in device memory.
struct LdsBlock {
    const uint32_t* B;
    int W;
    // word q of row p (empty below the row's own)
    __device__ __forceinline__ uint64_t word(int p, int q) const {
        const int g = p >> 6;
        if (q < g) return 0ull;
        const uint32_t* x = B + packed_base(g, W) + (p & 63) * packed_stride(g, W) + 2 * (q - g);
        return (uint64_t)x[0] | ((uint64_t)x[1] << 32);
    }
    __device__ __forceinline__ uint32_t dword(int p, int c) const { return PackedRows{B, W}.get(p >> 6, p & 63, c); }
};

struct DevBlock {
    const uint64_t* B;
    int W;
    __device__ __forceinline__ uint64_t word(int p, int q) const { return B[p * W + q]; }
    __device__ __forceinline__ uint32_t dword(int p, int c) const {
        return reinterpret_cast<const uint32_t*>(B)[p * 2 * W + c];
    }
};

// A block's rows cut to a set (lane c: dword c).
template <class Block>
struct CutRows {
    Block X;
    uint32_t sv;
    __device__ __forceinline__ uint32_t get(int q, int i, int c) const {
        const int p = 64 * q + i;
        const uint32_t rows = (uint32_t)__shfl((int)sv, p >> 5), cols = (uint32_t)__shfl((int)sv, c);
        return (rows >> (p & 31)) & 1u ? X.dword(p, c) & cols : 0u;
    }
};

using f32x16 = float __attribute__((ext_vector_type(16)));
using i32x8 = int32_t __attribute__((ext_vector_type(8)));

// 32 bits as 32 four-bit floats, 0 or 0.5, in the order of bits 0, 4, 8, ..,
// 1, 5, ..: the order is that of both operands, so the products meet.
__device__ __forceinline__ i32x8 as_fp4(uint32_t x) {
    i32x8 r = {0, 0, 0, 0, 0, 0, 0, 0};
    r[0] = (int32_t)(x & 0x11111111u);
    r[1] = (int32_t)((x >> 1) & 0x11111111u);
    r[2] = (int32_t)((x >> 2) & 0x11111111u);
    r[3] = (int32_t)((x >> 3) & 0x11111111u);
    return r;
}

// C += I J^T over 64 positions, in units of 2^-22 (the block scales of 2^-10 and the
// halves): started at 2, C's low 24 bits are a whole number (below 2^22).
__device__ __forceinline__ f32x16 mfma_bits(i32x8 I, i32x8 J, f32x16 C) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(I, J, C, 4, 4, 0, 0x75757575, 0, 0x75757575);
}

// Sum of C over the positions set in m, by products of 24 bits: C's lane l
// holds column l % 32 and rows 8 (v / 4) + 4 (l / 32) + v % 4; m is the lane's column,
// shifted by 4 (l / 32).
__device__ __forceinline__ uint32_t masked_sum(const f32x16& C, uint32_t m) {
    uint32_t t = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        uint32_t on = __builtin_amdgcn_ubfe(m, 8 * (v / 4) + v % 4, 1);
        // the value is hidden: known to be 0 or 1, the product becomes a compare, a
        // select and an add
        asm("" : "+v"(on));
        t += __umul24(__float_as_uint(C[v]), on);
    }
    return t;
}

// Triangles j < i < k with j in rows 64a .. and i in rows 64b .. (a <= b), of n
// rows in nw words: the lane's share.  Bound by the 40 instructions that take
// the sum over a tile of 32 x 32; a product adds 32 cycles per 64 positions.
template <class Rows>
__device__ __forceinline__ uint32_t triangles_block(const Rows& X, int a, int b, int nw, int n) {
    const int col = lane() & 31, half = lane() >> 5;
    const bool second = 64 * b + 32 < n;   // rows 32.. of b (if not, a's are full or a = b)
    uint32_t t = 0;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
        if (ti == 1 && !second) break;
        // rows j above those of i see none of them
        const bool both = a < b || ti == 1;
        f32x16 c0, c1;
        {
            const int c = 2 * b + half;
            const i32x8 I = as_fp4(X.get(b, 32 * ti + col, c));
            const f32x16 two = {2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f,
                                2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f, 2.0f};
            c0 = mfma_bits(I, as_fp4(X.get(a, col, c)), two);
            if (both) c1 = mfma_bits(I, as_fp4(X.get(a, 32 + col, c)), two);
        }
        for (int k = b + 1; k < nw; ++k) {
            const int c = 2 * k + half;
            const i32x8 I = as_fp4(X.get(b, 32 * ti + col, c));
            c0 = mfma_bits(I, as_fp4(X.get(a, col, c)), c0);
            if (both) c1 = mfma_bits(I, as_fp4(X.get(a, 32 + col, c)), c1);
        }
        t += masked_sum(c0, X.get(a, col, 2 * b + ti) >> (4 * half));
        if (both) t += masked_sum(c1, X.get(a, 32 + col, 2 * b + ti) >> (4 * half));
    }
    return t;
}

// Triangles among the positions s of one word, R the lane's row of that word.
__device__ __forceinline__ uint32_t triangles_word(uint64_t R, uint64_t s) {
    uint32_t c = 0;
    R &= s;
    uint64_t todo = s & ballot(R != 0ull);
    while (todo) {
        const int j = __builtin_ctzll(todo);
        todo &= todo - 1;
        const uint64_t t = readlane64(R, j);
        if (__builtin_amdgcn_inverse_ballot_w64(t)) c += (uint32_t)__popcll(R & t);
    }
    return c;
}

struct SetLds {
    uint32_t rows[packed_dwords(ST_N / 64)];
    uint16_t list[ST_N];
};

// Triangles among the set sv (lane c: dword c, empty from 2 W on) of a block's
// rows: the lane's share.
template <class Block>
__device__ __forceinline__ uint32_t triangles_set(uint32_t sv, const Block& X, SetLds& L) {
    const int W = X.W;
    auto word = [&](int q) {
        return (uint64_t)(uint32_t)readlane((int32_t)sv, 2 * q) |
               ((uint64_t)(uint32_t)readlane((int32_t)sv, 2 * q + 1) << 32);
    };
    const uint64_t nz = ballot(sv != 0u);
    const uint32_t words = (uint32_t)((nz | (nz >> 1)) & 0x555555ull);   // bit 2q: word q is not empty
    if (words == 0) return 0;
    if ((words & (words - 1)) == 0) {
        const int q = __builtin_ctz(words) >> 1;
        const uint64_t s = word(q);
        if (popc64(s) < 3) return 0;
        const uint64_t R = (s >> lane()) & 1ull ? X.word(64 * q + lane(), q) : 0ull;
        return triangles_word(R, s);
    }
    int n = 0;
    for (uint32_t t = words; t; t &= t - 1) {
        const int q = __builtin_ctz(t) >> 1;
        const uint64_t s = word(q);
        const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(s >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)s, 0u));
        if (((s >> lane()) & 1ull) && at < ST_N) L.list[at] = (uint16_t)(64 * q + lane());
        n += popc64(s);
    }
    uint32_t c = 0;
    if (n < 3) return 0;
    wave_sync();
    if (n > ST_N) {   // too many to pack
        const CutRows<Block> C{X, sv};
        for (int b = 0; b < W; ++b)
            for (int a = 0; a <= b; ++a) c += triangles_block(C, a, b, W, 64 * W);
        wave_sync();
        return c;
    }
    const int nw = (n + 63) >> 6;
    for (int g = 0; g < nw; ++g) {
        const int x = 64 * g + lane();
        const int p = L.list[x < n ? x : n - 1];
        uint32_t* out = L.rows + packed_base(g, nw) + lane() * packed_stride(g, nw);
        int k = 0;            // members seen
        uint64_t acc = 0;     // the row's bits from member k & ~31 on
        // 32 places of the row: its bits at the members among them are moved
        // together, a scalar loop over the members
        auto take = [&](uint32_t bits, uint32_t from) {
            if (!bits) return;
            uint32_t t = 0;
            const int i = __builtin_popcount(bits);
            int at = 0;
            if (i & 1) {
                t = __builtin_amdgcn_ubfe(from, __builtin_ctz(bits), 1);
                at = 1;
                bits &= bits - 1;
            }
            while (bits) {   // two a turn: the scalar instructions bound it
                const int p0 = __builtin_ctz(bits);
                bits &= bits - 1;
                const int p1 = __builtin_ctz(bits);
                bits &= bits - 1;
                t |= (__builtin_amdgcn_ubfe(from, p0, 1) | (__builtin_amdgcn_ubfe(from, p1, 1) << 1)) << at;
                at += 2;
            }
            acc |= (uint64_t)t << (k & 31);
            if ((k & 31) + i >= 32) {
                if ((k >> 5) >= 2 * g) out[(k >> 5) - 2 * g] = (uint32_t)acc;
                acc >>= 32;
            }
            k += i;
        };
        uint32_t t = words;
        int q = __builtin_ctz(t) >> 1;
        uint64_t r = x < n ? X.word(p, q) : 0ull;
        while (true) {
            t &= t - 1;
            const int q2 = t ? __builtin_ctz(t) >> 1 : q;
            const uint64_t r2 = x < n ? X.word(p, q2) : 0ull;   // flies during this word's loop
            take((uint32_t)readlane((int32_t)sv, 2 * q), (uint32_t)r);
            take((uint32_t)readlane((int32_t)sv, 2 * q + 1), (uint32_t)(r >> 32));
            if (!t) break;
            q = q2;
            r = r2;
        }
        // the rest of the last words
        for (int d = k >> 5; d < 2 * nw; ++d) {
            if (d >= 2 * g) out[d - 2 * g] = (uint32_t)acc;
            acc = 0;
        }
    }
    wave_sync();
    const PackedRows Y{L.rows, nw};
    for (int b = 0; b < nw; ++b)
        for (int a = 0; a <= b; ++a) c += triangles_block(Y, a, b, nw, n);
    wave_sync();   // read before the next set's
    return c;
}

__device__ __forceinline__ void add_count(uint64_t acc, unsigned long long* stats) {
    acc = wave_sum_u64(acc);
    if (lane() == 0) add_stat(stats, 0, acc);
}

}  // namespace

// k-cliques (k = 4, 5) at roots of at most 64 out-neighbours: a wave takes a run
// of roots (up to 64) and then, one by one, a row per lane.
template <int K>
__global__ __launch_bounds__(ST_THREADS) void k_small_root_sets(XcdQueue Q, const int32_t* __restrict__ roots,
                                                                const int64_t* __restrict__ rp,
                                                                const uint64_t* __restrict__ moff,
                                                                const uint64_t* __restrict__ M,
                                                                unsigned long long* __restrict__ stats) {
    uint64_t acc = 0;
    QueueCursor cur = queue_start();
    int64_t end = 0;
    for (int64_t it = queue_next(Q, cur, end); it >= 0; it = queue_next(Q, cur, end)) {
        int64_t base = 0;
        int D = 0;
        if (it + lane() < end) {
            const int32_t r = roots[Q.n_items - 1 - (it + lane())];   // wider roots first
            D = (int)(rp[r + 1] - rp[r]);
            base = (int64_t)moff[r];
        }
        uint64_t todo = ballot(D >= K - 1);
        uint64_t R = 0;
        auto load = [&](uint64_t left) {
            const int l = __builtin_ctzll(left);
            const int d = readlane(D, l);
            return lane() < d ? M[(int64_t)readlane64((uint64_t)base, l) + lane()] : 0ull;
        };
        if (todo) R = load(todo);
        while (todo) {
            todo &= todo - 1;
            const uint64_t next = todo ? load(todo) : 0ull;   // flies during this root's count
            if constexpr (K == 4) acc += triangles_word(R, ~0ull);
            else
                for (uint64_t t = ballot(popc64(R) >= 3); t; t &= t - 1)
                    acc += triangles_word(R, readlane64(R, __builtin_ctzll(t)));
            R = next;
        }
    }
    add_count(acc, stats);
}

// The rows of root r from group g0 on, packed in LDS: a power of two of threads
// per row.
__device__ __forceinline__ void stage_rows(uint32_t* rows, const uint64_t* __restrict__ blk, int D, int W, int g0) {
    const int lg = W <= 2 ? 1 : (W <= 4 ? 2 : (W <= 8 ? 3 : 4));
    for (int i = (int)threadIdx.x + ((64 * g0) << lg); i < (64 * W) << lg; i += (int)blockDim.x) {
        const int p = i >> lg, c = i & ((1 << lg) - 1), q = p >> 6;
        if (c < q || c >= W) continue;
        const uint64_t x = p < D ? blk[p * W + c] : 0ull;
        uint32_t* out = rows + packed_base(q, W) + (p & 63) * packed_stride(q, W) + 2 * (c - q);
        out[0] = (uint32_t)x;
        out[1] = (uint32_t)(x >> 32);
    }
}

// 4-cliques at wider roots: a workgroup stages the root's rows in LDS and its
// waves take pairs of row blocks.
__global__ __launch_bounds__(ST_THREADS, 4) void k_wide_root_sets(XcdQueue Q, const int32_t* __restrict__ roots,
                                                                  const int64_t* __restrict__ rp,
                                                                  const uint64_t* __restrict__ moff,
                                                                  const uint64_t* __restrict__ M,
                                                                  unsigned long long* __restrict__ stats) {
    extern __shared__ uint32_t rows[];
    __shared__ int64_t s_item;
    const int w = threadIdx.x / WAVE;
    uint64_t acc = 0;
    QueueCursor cur = queue_start(1);
    while (true) {
        __syncthreads();   // the previous root's rows are read
        if (w == 0) {
            int64_t end = 0;
            const int64_t it = queue_next(Q, cur, end);
            if (lane() == 0) s_item = it;
        }
        __syncthreads();
        const int64_t it = uniform64(s_item);
        if (it < 0) break;
        const int32_t r = roots[Q.n_items - 1 - it];
        const int D = (int)(rp[r + 1] - rp[r]);
        const int W = (D + 63) >> 6;
        const uint64_t* blk = M + moff[r];
        stage_rows(rows, blk, D, W, 0);
        __syncthreads();
        const PackedRows X{rows, W};
        int turn = 0;
        for (int b = 0; b < W; ++b)
            for (int a = 0; a <= b; ++a)
                if ((turn++ & (ST_WAVES - 1)) == w) acc += triangles_block(X, a, b, W, D);
    }
    add_count(acc, stats);
}

// 5-cliques at wider roots: a workgroup stages the root's rows in LDS (from the
// item's first entry on: an entry's set lies above it) and its waves take the
// entries one by one.  An item is a root, or 64 entries of it.
__global__ __launch_bounds__(2 * ST_THREADS, 5) void k_wide_entry_sets(XcdQueue Q, const int32_t* __restrict__ roots,
                                                                      int parts, const int64_t* __restrict__ rp,
                                                                      const uint64_t* __restrict__ moff,
                                                                      const uint64_t* __restrict__ M,
                                                                      unsigned long long* __restrict__ stats) {
    extern __shared__ uint32_t shared[];   // a SetLds per wave, then the block
    __shared__ int64_t s_item;
    __shared__ int32_t s_entry;
    const int w = threadIdx.x / WAVE;
    SetLds& L = reinterpret_cast<SetLds*>(shared)[w];
    uint32_t* rows = reinterpret_cast<uint32_t*>(reinterpret_cast<SetLds*>(shared) + blockDim.x / WAVE);
    uint64_t acc = 0;
    QueueCursor cur = queue_start(1);
    while (true) {
        __syncthreads();   // the previous item's rows are read
        if (w == 0) {
            int64_t end = 0;
            const int64_t it = queue_next(Q, cur, end);
            if (lane() == 0) s_item = it;
        }
        __syncthreads();
        const int64_t it = uniform64(s_item);
        if (it < 0) break;
        const int32_t r = uniform(roots[Q.n_items / parts - 1 - it / parts]);
        const int part = (int)(it % parts);
        const int D = uniform((int32_t)(rp[r + 1] - rp[r]));
        const int W = (D + 63) >> 6;
        if (part >= W) continue;
        // the last three entries have no set of three
        const int x1 = parts == 1 ? D - 3 : min(64 * part + 64, D - 3);
        if (threadIdx.x == 0) s_entry = 64 * part;
        stage_rows(rows, M + moff[r], D, W, part);
        __syncthreads();
        const LdsBlock X{rows, W};
        while (true) {
            int x = 0;
            if (lane() == 0) x = atomicAdd(&s_entry, 1);
            x = uniform(x);
            if (x >= x1) break;
            const uint32_t sv = lane() < 2 * W && lane() >= 2 * (x >> 6) ? X.dword(x, lane()) : 0u;
            acc += triangles_set(sv, X, L);
        }
    }
    add_count(acc, stats);
}

struct SetArgs {
    XcdQueue Q;                  // over entries of level lev
    int lev;
    MaskChain ch;
    const uint64_t* info;        // row_info of each level-1 entry
    const uint64_t* M;
    unsigned long long* stats;
};

// Cliques below the entries of a level lev >= 2: the triangles in each entry's
// set, the AND of the rows of its vertices after the root.  A wave forms the sets
// of 16 entries side by side (four lanes each: lane j of the four forms words j,
// j + 4 and j + 8) and then takes them one by one.
__global__ __launch_bounds__(ST_THREADS, 4) void k_entry_sets(SetArgs A) {
    __shared__ SetLds lds[ST_WAVES];
    __shared__ uint32_t sets[ST_WAVES][ST_PART][2 * BM_W];
    const int w = threadIdx.x / WAVE;
    const int sub = lane() & 3;
    uint64_t acc = 0;
    QueueCursor cur = queue_start();
    int64_t end = 0;
    for (int64_t it = queue_next(A.Q, cur, end); it >= 0; it = queue_next(A.Q, cur, end)) {
        uint64_t sp[BM_W / 4] = {0ull, 0ull, 0ull};
        int W = 0;               // of the lane's entry
        int64_t bl = 0;
        int64_t c = it + lane() / 4;
        if (c < end) {
            int32_t apos[PG_KMAX];
            int na = 0;
            for (int l = A.lev; l >= 2; --l) {
                apos[na++] = A.ch.pos[l][c];
                c = A.ch.idx[l][c];
            }
            const uint64_t f = A.info[c];   // c: the level-1 entry
            W = info_w(f);
            bl = (int64_t)info_base(f);
            const uint64_t* blk = A.M + bl;
#pragma unroll
            for (int q = 0; q < BM_W / 4; ++q)
                if (4 * q + sub < W) sp[q] = blk[(int64_t)info_i(f) * W + 4 * q + sub];
            for (int a = 0; a < na; ++a)
#pragma unroll
                for (int q = 0; q < BM_W / 4; ++q)
                    if (4 * q + sub < W) sp[q] &= blk[(int64_t)apos[a] * W + 4 * q + sub];
        }
        uint64_t todo = ballot((sp[0] | sp[1] | sp[2]) != 0ull);
#pragma unroll
        for (int q = 0; q < BM_W / 4; ++q) {
            sets[w][lane() / 4][2 * (4 * q + sub)] = (uint32_t)sp[q];
            sets[w][lane() / 4][2 * (4 * q + sub) + 1] = (uint32_t)(sp[q] >> 32);
        }
        wave_sync();
        while (todo) {
            const int l0 = __builtin_ctzll(todo) & ~3;
            todo &= ~(15ull << l0);
            const DevBlock X{A.M + (int64_t)readlane64((uint64_t)bl, l0), readlane(W, l0)};
            acc += triangles_set(lane() < 2 * X.W ? sets[w][l0 / 4][lane()] : 0u, X, lds[w]);
        }
        wave_sync();   // the sets are read before the next entries'
    }
    add_count(acc, A.stats);
}

static XcdQueue set_queue(unsigned long long* next, int64_t n_items, int64_t chunk) {
    XcdQueue Q;
    Q.next = next;
    Q.n_items = n_items;
    Q.chunk = chunk;
    return Q;
}

void count_root_sets(pg_graph* g, int k, const uint64_t* M, unsigned long long* queues, unsigned long long* stats) {
    const MaskPlan& P = g->dag.plan;
    hipStream_t s = g->stream;
    const int64_t* rp = g->dag.rp.as<int64_t>();
    const uint64_t* moff = P.moff.as<uint64_t>();
    ProfScope ps("clique_last", s, 0.0);
    for (int c = CQ_CLASSES - 1; c >= 0; --c) {   // the most work first
        const int64_t n = P.n_roots[c];
        if (n == 0) continue;
        const int32_t* roots = P.roots[c].as<int32_t>();
        unsigned long long* queue = queues + c * Q_WORDS;
        if (CQ_CLASS_MAX[c] <= 64) {
            // a few hundred instructions per root of the lower class: up to 32 a
            // turn; some thousands (k = 5: tens of thousands) in the upper one
            const int most = c == 0 ? 32 : (k == 4 ? 8 : 4);
            const auto kernel = k == 4 ? k_small_root_sets<4> : k_small_root_sets<5>;
            const unsigned blocks = queue_blocks(kernel, ST_THREADS, 0, (n + ST_WAVES - 1) / ST_WAVES);
            const int64_t waves = (int64_t)blocks * ST_WAVES;
            const int64_t chunk = queue_chunk(n, waves, most);
            kernel<<<blocks, ST_THREADS, 0, s>>>(set_queue(queue, n, chunk), roots, rp, moff, M, stats);
        } else {
            const int W = (int)((std::min<int64_t>(g->dag.max_out, CQ_CLASS_MAX[c]) + 63) / 64);
            const size_t block = sizeof(uint32_t) * packed_dwords(W);
            if (k == 4) {
                const unsigned blocks = queue_blocks(k_wide_root_sets, ST_THREADS, block, n);
                k_wide_root_sets<<<blocks, ST_THREADS, block, s>>>(
                    set_queue(queue, n, queue_chunk(n, blocks, 1)), roots, rp, moff, M, stats);
            } else {
                // wider blocks leave room for fewer workgroups: these have more waves
                const int threads = c == 2 ? ST_THREADS : 2 * ST_THREADS;
                const size_t lds = sizeof(SetLds) * (threads / WAVE) + block;
                // a root at a time, or 64 entries where the roots would not fill the chip evenly
                if (lds > 64 * 1024)
                    PG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_wide_entry_sets),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
                const unsigned blocks = queue_blocks(k_wide_entry_sets, threads, lds, n * W);
                const int parts = n >= 8 * (int64_t)blocks ? 1 : W;
                k_wide_entry_sets<<<blocks, threads, lds, s>>>(
                    set_queue(queue, n * parts, queue_chunk(n * parts, blocks, 1)), roots, parts, rp, moff, M, stats);
            }
        }
        PG_HIP(hipGetLastError());
    }
}

void count_parent_sets(pg_graph* g, int lev, int64_t m, const MaskChain& ch, const uint64_t* info, const uint64_t* M,
                       unsigned long long* qctr, unsigned long long* stats) {
    if (m <= 0) return;
    hipStream_t s = g->stream;
    SetArgs A{};
    fill_u64(reinterpret_cast<uint64_t*>(qctr), Q_WORDS, 0, s);
    A.Q = set_queue(qctr, m, ST_PART);
    A.lev = lev;
    A.ch = ch;
    A.info = info;
    A.M = M;
    A.stats = stats;
    ProfScope ps("clique_last", s, 0.0);
    k_entry_sets<<<queue_blocks(k_entry_sets, ST_THREADS, 0, (m + ST_PART - 1) / ST_PART), ST_THREADS, 0, s>>>(A);
    PG_HIP(hipGetLastError());
}

}  // namespace pg
