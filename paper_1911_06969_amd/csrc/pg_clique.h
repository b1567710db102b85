// Sibling mask rows of the clique kernels, shared by the passes that write and
// read them.
//
// The out-list of a root r of the degree-ordered DAG, out(r), has at most
// BM_MAXD vertices at a light root.  Row i of r's block is the set of positions
// j of out(r) whose vertex is an out-neighbour of out(r)[i] (all above i), in
// W = ceil(out-degree / 64) words.
#pragma once

#include <stdint.h>

#include "pg_device.h"
#include "pg_internal.h"

namespace pg {

constexpr int BM_MAXD = 768;             // roots with out-degree up to this use masks
constexpr int BM_W = BM_MAXD / 64;       // 64-bit words per mask row

// Light roots by out-degree, for the last levels: [3, 16], (16, 64], (64, 256]
// and (256, 768].  Up to 64 a row is one word and a wave takes a root, a row per
// lane (the second class a root at a time, the first, of little work each, in
// runs).  Above, a workgroup stages the rows in LDS: 6 KB for the third class, up
// to 43 KB for the last.
constexpr int CQ_CLASSES = 4;
constexpr int CQ_CLASS_MAX[CQ_CLASSES] = {16, 64, 256, BM_MAXD};

constexpr int CLIQUE_QUEUES = 3 + CQ_CLASSES;       // work queues of a call of k <= 5

// Count-pass items by how elements are looked up: a table of 32 ids per entry
// over the root's list, in LDS (a small one, of which seven workgroups' fit a CU,
// or a large one, three), or a search of the list.  Below CR_MIN_D a search takes
// at most five steps and an item has too little to stream to pay for a
// workgroup's table: searches there took 1.2 ms of the 4-clique count of R-MAT
// scale 21, edge factor 13, for an eighth of the elements.
constexpr int CR_MIN_D = 32;                       // out-degree from which a table is laid out
constexpr int CR_WORDS[2] = {2560, 6400};          // 32 ids each
struct CountArgs {
    const int64_t* rp;          // DAG
    const int32_t* col;
    const uint64_t* moff;       // first mask word of each root
    uint64_t* M;                // mask rows; NULL: triangles are counted only
    uint32_t* count;            // children of each level-1 entry (with info; NULL: not wanted)
    uint64_t* info;             // row_info of each level-1 entry
    unsigned long long* stats;  // [0] += triangles when M is NULL, [3] += out-list entries streamed
    int round;                  // level-1 entries per item (64 or 16)
};

// Rows (or triangles) of the items of table class c, the count pass of these items.
// `queue`: Q_WORDS zeroed words.
void count_rows_table(pg_graph* g, int c, const CountArgs& A, unsigned long long* queue);

// Level-1 entry e = (r, S[i]) is described by one word: the first mask word
// of r's block, i, and the row width W (words):  base << 14 | i << 4 | W.
__host__ __device__ constexpr uint64_t row_info(uint64_t base, int i, int W) {
    return (base << 14) | ((uint64_t)i << 4) | (uint64_t)W;
}
__device__ __forceinline__ int info_w(uint64_t info) { return (int)(info & 15); }
__device__ __forceinline__ int info_i(uint64_t info) { return (int)((info >> 4) & 1023); }
__device__ __forceinline__ uint64_t info_base(uint64_t info) { return info >> 14; }

constexpr int BM_UNROLL = 4;             // out-list elements per lane per step (double-buffered)

// Streams out(v) of a level-1 entry (left > 0 elements from cp): BM_UNROLL loads
// per lane per step, double-buffered (the next step's loads fly during this step's
// look-up, the two buffers alternate).  look(u, n) takes the first n rows of 64
// elements of a step and returns the number of hits; the sum is returned
// (wave-uniform).  Stops once the list passes s_last.
//
// A step is read through a buffer descriptor over its valid elements: the
// address arithmetic is scalar, and lanes past the end read 0, which is
// never in out(r) (it holds ranks above r, so its elements are at least 1).
// Every step issues its loads (after the final step they repeat its first
// element), so the number of loads in flight is known at compile time and
// the look-up waits for its own step's data only.
template <class Look>
__device__ __forceinline__ uint32_t stream_list(const int32_t* cp, int64_t left, int32_t s_last, uint64_t& streamed,
                                                Look look) {
    constexpr int STEP = WAVE * BM_UNROLL;
    uint32_t c = 0;
    int32_t ua[BM_UNROLL], ub[BM_UNROLL];
    int32_t la = 0, lb = 0;   // valid elements of each buffer (wave-uniform)
    // lim >= 1 elements valid from p
    auto load = [&](int32_t (&u)[BM_UNROLL], const int32_t* p, int32_t lim) {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(p), (short)0, lim * 4, BUF_WORD3);
#pragma unroll
        for (int q = 0; q < BM_UNROLL; ++q)
            u[q] = __builtin_amdgcn_raw_buffer_load_b32(rs, (q * WAVE + lane()) * 4, 0, 0);
    };
    // A step is sorted: once the first key of a row of 64 exceeds s_last
    // (or the row is past the list), no key of it or of a later row hits.
    static_assert(BM_UNROLL == 4, "the row cases below are written out for four rows");
    auto search = [&](const int32_t (&u)[BM_UNROLL], int32_t lim) {
        auto live = [&](int q) { return q * WAVE < lim && readlane(u[q], 0) <= s_last; };
        if (live(3)) c += look(u, 4);
        else if (live(2)) c += look(u, 3);
        else if (live(1)) c += look(u, 2);
        else if (live(0)) c += look(u, 1);
    };
    // the next step's loads: of cp + STEP if there is one, else of cp again
    auto next = [&](int32_t (&u)[BM_UNROLL], int32_t& lim, bool more) {
        lim = more ? (int32_t)min64(left - STEP, STEP) : 1;
        load(u, more ? cp + STEP : cp, lim);
    };
    la = (int32_t)min64(left, STEP);
    load(ua, cp, la);
    while (true) {
        // ua holds the current step; ub gets the next one
        bool more = left > STEP && readlane(ua[BM_UNROLL - 1], WAVE - 1) <= s_last;
        next(ub, lb, more);
        search(ua, la);
        streamed += (uint64_t)min64(left, STEP);
        if (!more) break;
        cp += STEP;
        left -= STEP;
        // ub holds the current step; ua gets the next one
        more = left > STEP && readlane(ub[BM_UNROLL - 1], WAVE - 1) <= s_last;
        next(ua, la, more);
        search(ub, lb);
        streamed += (uint64_t)min64(left, STEP);
        if (!more) break;
        cp += STEP;
        left -= STEP;
    }
    return c;
}

// The stored levels an entry's ancestry is walked through.
struct MaskChain {
    const int32_t* idx[PG_KMAX + 1];    // level l >= 2: parent index (level 2: level-1 entry)
    const uint16_t* pos[PG_KMAX + 1];   // level l >= 2: position in the root's out-list
};

// Adds the k-cliques (k = 4, 5) at the light roots to stats[0], from their rows
// M.  `queues`: CQ_CLASSES * Q_WORDS zeroed words.
void count_root_sets(pg_graph* g, int k, const uint64_t* M, unsigned long long* queues, unsigned long long* stats);

// Adds to stats[0] the cliques of lev + 3 vertices below the entries [0, m) of
// level lev >= 2.
void count_parent_sets(pg_graph* g, int lev, int64_t m, const MaskChain& ch, const uint64_t* info, const uint64_t* M,
                       unsigned long long* qctr, unsigned long long* stats);

}  // namespace pg
