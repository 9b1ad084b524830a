// Sorting a batched run's points by host leaf (point_sort.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>

#include "ot_common.h"

namespace ot {

// Two sets of buffers the passes alternate between (set 1 after the first
// pass, set 0 after the second), plus the counting workspace.
template <typename T>
struct PointSortBufs {
    uint64_t *kv[2];   // n words: host's leaf entry (or block key) << 32 | input index
    T *rec[2];         // n records of 6 (position, force) or 3 (position) values
    void *ws;          // point_sort_ws_bytes(n)
};

template <typename T>
struct PointSortResult {
    const uint64_t *kv;   // per sorted position: host's leaf entry (or block key) << 32 | input index
    const T *rec;         // per sorted position: stride values, position first
    int stride;           // 6 with forces, 3 without
};

// Of exactly the n that is sorted: fewer points can make more tiles.
int64_t point_sort_ws_bytes(int64_t n);

// Memory the key launch clears for the kernels after it: `words` 32-bit words
// at p (a spreading target or workspace, or none), and a plan's counters.
struct SortZero {
    uint32_t *p;
    int64_t words;
    unsigned *counters;
    int n_counters;
};

// What a sort orders by: bits [shift, shift + bits) of a key, and the key of
// a point without a host (`none`, which sorts last).
struct PointSortKey {
    bool blocks;     // block keys (block_pass.h) instead of host leaf ids
    int shift, bits;
    uint32_t none;
};

// Host leaf ids (keys run up to n_leaves): groups of at most 64 consecutive
// leaf ids, and all of the id when it has at most 16 bits.  Trees of up to 4
// M leaves take two 8-bit passes, larger ones three (measured on 17 M and 20
// M leaves: groups of 512 leaves left a tile's points spread over more leaves
// than the spreading table holds; 64 beat 8 and 2 as well).
inline PointSortKey point_sort_by_host(int64_t n_leaves)
{
    int all = 1;
    while ((int64_t(1) << all) <= n_leaves) ++all;
    const int shift = std::max(0, std::min(6, all - 16));
    return {false, shift, all - shift, (uint32_t)n_leaves};
}

// Blocks (keys run up to nblk): every key bit.
inline PointSortKey point_sort_by_block(int32_t nblk)
{
    int all = 1;
    while ((int64_t(1) << all) <= nblk) ++all;
    return {true, 0, all, (uint32_t)nblk};
}

// Keys, ids when ids != null, then ceil(bits / 8) passes (all stable but the
// first) over the key bits; bits >= 1.  The sorted words hold the host's leaf
// entry (id in the low 26 bits), or the block key.  force != null: records
// carry forces too, and when maxbits != null the first pass also atomically
// maxes the bit pattern of max |F| (finite components) into maxbits[0] and
// sets maxbits[1] when a component is not finite.
template <typename T>
void point_sort(const TreeView &tv, int64_t n, const PointSortKey &key, const T *pos, const T *force, int32_t *ids,
                PointSortBufs<T> &b, const SortZero &zero, unsigned long long *maxbits, hipStream_t s,
                PointSortResult<T> &out);

}  // namespace ot
