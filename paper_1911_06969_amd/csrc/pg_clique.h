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

constexpr int ROW_QUEUES = 3;                       // work queues of the count pass
constexpr int CLIQUE_QUEUES = ROW_QUEUES + CQ_CLASSES;   // of a call of k <= 5

struct CountArgs {
    const int64_t* rp;          // DAG
    const int32_t* col;
    const int64_t* in_rp;       // in-lists: edges (r, v) by v
    const int32_t* in_edge;
    const int32_t* in_src;      // r
    const uint64_t* moff;       // first mask word of each root
    uint64_t* M;                // mask rows, zeroed; NULL: triangles are counted only
    uint32_t* count;            // children of each level-1 entry, zeroed (NULL: not wanted)
    uint64_t* info;             // row_info of each level-1 entry with children (NULL: not wanted)
    unsigned long long* stats;  // [0] += triangles when M is NULL, [3] += out-list entries read
};

// The count pass's items, and the DAG's in-lists if they are not made yet (part of the
// plan of a graph).  Returns the last words of moff and hrp with them.
void build_in_lists(pg_graph* g, uint64_t* moff_total, uint64_t* heavy_total);

// The count pass: rows (or triangles) of the light roots.  A: M, count, info and
// stats are set.  `queues`: ROW_QUEUES * Q_WORDS zeroed words.
void count_rows(pg_graph* g, CountArgs A, unsigned long long* queues);

// Level-1 entry e = (r, S[i]) is described by one word: the first mask word
// of r's block, i, and the row width W (words):  base << 14 | i << 4 | W.
__host__ __device__ constexpr uint64_t row_info(uint64_t base, int i, int W) {
    return (base << 14) | ((uint64_t)i << 4) | (uint64_t)W;
}
__device__ __forceinline__ int info_w(uint64_t info) { return (int)(info & 15); }
__device__ __forceinline__ int info_i(uint64_t info) { return (int)((info >> 4) & 1023); }
__device__ __forceinline__ uint64_t info_base(uint64_t info) { return info >> 14; }

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
