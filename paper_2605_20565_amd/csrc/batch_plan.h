// State of a batched plan (ot_batch_plan), shared by the plan's host code
// (batch.hip) and its kernels' enqueue sequence (batch_kernels.h).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "ot_common.h"
#include "point_sort.h"

namespace ot {
struct BlkTile;
// Device memory of a run's block pass (block_pass.h): work words (counts and
// queues), tiles of root cubes and of sub-tables, and the sparse blocks'
// ranges (first sorted point, count).
struct BlkWork {
    int64_t n;               // points
    unsigned *words;
    BlkTile *root_tiles, *sub_tiles;
    uint2 *ranges;
    int grid;                // persistent workgroups of each pass
};
int64_t blk_bytes(const ot_tree *t, int64_t n);       // device bytes besides the words
int64_t blk_tile_pts(const ot_tree *t, int64_t n);    // most points of a tile
void blk_layout(const ot_tree *t, int64_t n, void *mem, unsigned *words, BlkWork *w);
// The pass over sorted points: tiles of blocks, short ranges, or neither (tiles
// of points sorted by host); wide: FP32 sums kept in FP64 (ot_batch_plan::wide).
struct SortedRoute {
    bool blocks, nodes, wide;
};
SortedRoute sorted_route(const ot_tree *t, int64_t n, int ops, int dtype, int mode, bool plan);
bool plain_sorts(const ot_tree *t, int64_t n, int ops, int dtype, int mode);   // a plain call's points
// whether a sorted plan takes the unsorted passes of plain calls
bool small_rule(const ot_tree *t, int64_t n, int ops, int dtype, int mode);
// plain calls that spread sort from here on (track.hip)
constexpr int64_t kSortMinSpread = 55000, kSortMinF32Sums = 30000, kSortMinF64Both = 65536;
constexpr int64_t kFewLeaves = 512;   // a tree that the smallest spreading table holds (track.hip)
}  // namespace ot

struct ot_batch_plan {
    const ot_tree *tree;
    int dtype, mode;
    int block, tile, grid;
    int ops_union;
    int64_t n_points, n_tiles;
    int64_t *tile_start;      // device
    uint32_t *tile_info;      // device: count | ops << 24
    unsigned *counter;        // device
    hipStream_t capture_stream;
    bool use_graph;           // OT_TUNE_GRAPH: runs replay a captured graph
    bool have_graph;
    hipGraph_t graph;
    hipGraphExec_t exec;
    const void *key[7];
    bool timing;              // record ev[0]/ev[1] around the persistent kernel
    hipEvent_t ev[2];
    // point sorting (OT_TUNE_SORT_POINTS)
    bool sort_points;
    ot::PointSortKey sort_key;
    int ops_all;              // the common ops of every instance
    bool grad_plan;           // instances carry OT_OP_GRAD_POS
    bool small_table;         // tiles of at most kSmallTile points: the small spreading table
    uint64_t *skv[2];         // host's leaf entry << 32 | input index, in sorted order
    void *srec[2];            // position (+ force) records in sorted order
    void *sws;                // counting workspace
    void *fxws;               // spreading workspace (FIXED plans that spread, and wide ones)
    int accumulate;           // add to field_out (plain calls)
    bool use_blocks;          // block pass
    bool use_small;           // unsorted passes of a plain call
    bool use_nodes;           // node-parallel pass over all sorted points
    // FP32 ATOMIC sums kept in FP64 until the end of the run: the passes over
    // blocks and short ranges add more often to a leaf than whole tiles of sorted
    // points do, and each add to FP32 rounds (relative error of a spread field, 40 k
    // points on 4,096 leaves: 1.3e-7 by tiles, 3.0e-7 with adds to FP32).
    bool wide;
    ot::BlkWork blk;
    void *blk_mem;
    // host-major pass (sorted forward plans with OT_TUNE_HOST_MAJOR)
    bool use_hm;
    int hm_grid;
    int64_t n_win;            // windows of kHmThreads sorted points
    uint32_t *fb_list;        // device: windows handed to the per-point pass
};

namespace ot {
constexpr uint32_t kCountMask = 0x00FFFFFFu;   // tile_info: point count in the low 24 bits
}  // namespace ot
