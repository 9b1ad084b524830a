// Host side of the block pass (block_pass.h): its device memory and the rule
// that chooses it.
#include <algorithm>

#include "batch_plan.h"
#include "block_pass.h"

namespace ot {

// Points per tile: whole blocks in large runs, and in smaller ones short tiles
// for two workgroups per CU (a tile of 2,000 points takes ~50 us alone).
int64_t blk_tile_pts(const ot_tree *t, int64_t n)
{
    return std::min<int64_t>(kBlkTilePts, std::max<int64_t>(kBlkTileMin, n / (2 * t->cus)));
}

namespace {
int64_t align256(int64_t b) { return (b + 255) & ~int64_t(255); }
// a dense block of c points gets ceil(c / blk_tile_pts) tiles; a run of sparse
// blocks ends at a dense block or at the end of a workgroup's keys
int64_t max_tiles(int64_t n) { return n / kBlkDense + n / kBlkTileMin + 1; }

int64_t max_ranges(const ot_tree *t, int64_t n)
{
    return n / kBlkWindow + n / kBlkDense + (int64_t)t->view.nblk / 64 + 4;
}

// The blocks among the sorted words, and the passes' work: tiles of the blocks
// with enough points (root cubes and sub-tables apart), and ranges of at most
// kBlkWindow points for the node-parallel pass (sparser blocks next to each other
// in the order, and points without a host).  A workgroup takes kBlkKeys - 1
// consecutive keys; eight lanes find a key's first point, probing eight places
// of the remaining range at once, so a search is ~log_9 n dependent loads.
constexpr int kBlkKeys = 128;
__global__ __launch_bounds__(kBlkKeys * 8) void k_block_bounds(TreeView tv, const uint64_t *__restrict__ kv, int64_t n,
                                                               uint32_t tile_pts, unsigned *__restrict__ words,
                                                               BlkTile *__restrict__ root_tiles,
                                                               BlkTile *__restrict__ sub_tiles,
                                                               uint2 *__restrict__ ranges)
{
    __shared__ uint32_t st[kBlkKeys];
    __shared__ uint64_t sparse[kBlkKeys / 64];
    __shared__ unsigned cnt[3], base[3];   // root tiles, sub-table tiles, ranges
    const uint32_t nblk = (uint32_t)tv.nblk, blk1 = (uint32_t)tv.blk1;
    const int grp = threadIdx.x >> 3, sub = threadIdx.x & 7, seg = (threadIdx.x & 63) & ~7;
    const uint32_t key = blockIdx.x * (uint32_t)(kBlkKeys - 1) + (uint32_t)grp;
    if (threadIdx.x < 3) cnt[threadIdx.x] = 0u;
    // keys run up to nblk (no host); nblk + 1 starts at n
    int64_t lo = key > nblk ? n : 0, hi = n;
    while (__any(lo < hi)) {
        const int64_t p = lo + (hi - lo) * (sub + 1) / 9;
        const bool less = lo < hi && ((uint32_t)(kv[p] >> 32) & kIdMask) < key;
        const unsigned m = (unsigned)(__ballot(less) >> seg) & 255u;
        if (lo < hi) {
            const int c = __popc(m);
            const int64_t l = lo, len = hi - lo;
            if (c > 0) lo = l + len * c / 9 + 1;
            if (c < 8) hi = l + len * (c + 1) / 9;
        }
    }
    if (sub == 0) st[grp] = (uint32_t)lo;
    __syncthreads();
    // one thread per key from here on
    const int g = (int)threadIdx.x;
    const uint32_t k = blockIdx.x * (uint32_t)(kBlkKeys - 1) + (uint32_t)g;
    const bool mine = g < kBlkKeys - 1 && k <= nblk;
    const uint32_t s = mine ? st[g] : 0u, c = mine ? st[g + 1] - s : 0u;
    const int which = k < blk1 ? 0 : 1;
    const bool dense = mine && k < nblk && c >= (uint32_t)kBlkDense;
    if (g < kBlkKeys) {
        const uint64_t b = __ballot(mine && !dense);
        if ((g & 63) == 0) sparse[g >> 6] = b;
    }
    __syncthreads();
    uint32_t nt = 0, nr = 0, at = 0, rs = 0, re = 0;
    if (dense) {
        nt = (c + tile_pts - 1) / tile_pts;
        at = atomicAdd(&cnt[which], nt);
    } else if (mine && (g == 0 || !((sparse[(g - 1) >> 6] >> ((g - 1) & 63)) & 1ull))) {
        // the first of consecutive sparse keys takes the points of all of them
        int e = g;   // the run's last key
        const uint64_t z0 = ~sparse[0], z1 = ~sparse[1];
        const uint64_t f0 = g < 64 ? z0 >> g : 0ull;
        if (f0) e = g + __ffsll((unsigned long long)f0) - 1;
        else {
            const int h = g < 64 ? 0 : g - 64;
            const uint64_t f1 = z1 >> h;
            e = f1 ? 64 + h + __ffsll((unsigned long long)f1) - 1 : kBlkKeys;
        }
        rs = s;
        re = st[min(e, kBlkKeys - 1)];
        nr = (re - rs + kBlkWindow - 1) / kBlkWindow;
        if (nr) at = atomicAdd(&cnt[2], nr);
    }
    __syncthreads();
    if (threadIdx.x < 3)
        base[threadIdx.x] = cnt[threadIdx.x] ? atomicAdd(&words[kBlkRootTiles + threadIdx.x], cnt[threadIdx.x]) : 0u;
    __syncthreads();
    if (nt) {
        BlkTile *out = (which ? sub_tiles : root_tiles) + base[which] + at;
        // the block's cell, its level l0 and the levels d below it
        int l0 = tv.lev[0] - kBlkBits, d = kBlkBits;
        uint64_t m = k;
        if (which) {
            int u = 1;
            while (u + 1 < tv.nlev && (int64_t)k >= tv.blk_base[u + 1]) ++u;
            l0 = min(tv.lev[0] + 3 * (u - 1), tv.L);
            d = min(tv.lev[0] + 3 * u, tv.L) - l0;
            m = tv.blk_anchor[k - blk1] >> (3 * (tv.L - l0));
        }
        const uint32_t a[3] = {compact3_21(m), compact3_21(m >> 1), compact3_21(m >> 2)};
        for (uint32_t i = 0; i < nt; ++i) {
            const uint32_t b = (uint32_t)((uint64_t)c * i / nt), e = (uint32_t)((uint64_t)c * (i + 1) / nt);
            out[i] = BlkTile{s + b, e - b, k, l0, {a[0], a[1], a[2]}, d};
        }
    }
    for (uint32_t i = 0; i < nr; ++i)
        ranges[base[2] + at + i] = make_uint2(rs + i * kBlkWindow, min((uint32_t)kBlkWindow, re - rs - i * kBlkWindow));
}

}  // namespace

void enqueue_bounds(const ot_tree *t, BlkWork &w, const uint64_t *kv, hipStream_t s)
{
    const TreeView &tv = t->view;
    const unsigned nb = (unsigned)((tv.nblk + kBlkKeys - 1) / (kBlkKeys - 1));   // keys 0 .. nblk
    hipLaunchKernelGGL(k_block_bounds, dim3(nb), dim3(kBlkKeys * 8), 0, s, tv, kv, w.n,
                       (uint32_t)blk_tile_pts(t, w.n), w.words, w.root_tiles, w.sub_tiles, w.ranges);
}

int64_t blk_bytes(const ot_tree *t, int64_t n)
{
    return 2 * align256((int64_t)sizeof(BlkTile) * max_tiles(n)) + align256(8 * max_ranges(t, n));
}

void blk_layout(const ot_tree *t, int64_t n, void *mem, unsigned *words, BlkWork *w)
{
    char *p = (char *)mem;
    w->n = n;
    w->grid = 2 * t->cus;   // as many as fit in FP32; later ones find the queue empty
    w->words = words;
    w->root_tiles = (BlkTile *)p;
    p += align256((int64_t)sizeof(BlkTile) * max_tiles(n));
    w->sub_tiles = (BlkTile *)p;
    p += align256((int64_t)sizeof(BlkTile) * max_tiles(n));
    w->ranges = (uint2 *)p;
}

// The pass over sorted points.
//
// Blocks.  Root cubes need a root of at least 8^3 cells.  Fewer than 64 points
// per block on average, or fewer than one per three leaves, leave most blocks to
// the short ranges or make tiles that cost more than their points: 600 k random
// points on 2.7 M leaves take 365 us, ranges 304, tiles of points sorted by host
// 329 (1 M: 307, 298, 352; markers 188, 243, 224).  The pass has three launches
// more than the others.  Spreading, FP32, ranges against blocks: 200 k points on
// 38 k leaves 91 against 117 us, 400 k 126 and 144, 600 k 162 and 159, 1 M 209 and
// 168; on 0.6 M leaves 400 k 143 and 167, 1 M 217 and 208; markers on 38 k leaves
// 331 k points 115 against 126, FP64 128 and 148, and with interpolation, whose
// values ranges must buffer in LDS, 137 against 136 and 190 against 163.
//
// Ranges are a short chain where tiles of points sorted by host are a long one
// (200 k points on 38 k leaves 91 us against 116), but each looks its nodes up
// anew, and in FP64 with gathers one workgroup fills a CU's LDS: forward and
// backward of 200 k points FP64 on 38 k leaves 150 us and 128 by tiles, 300 k on
// 0.6 M leaves 215 and 163, 600 k on 2.7 M leaves 466 and 387 (spreading 326 and
// 374).  Points much rarer than leaves share nothing in a tile (300 k on 17 M
// leaves 413 and 574 us; 4 M 1585 and 1135).
constexpr int64_t kBlkMinSpread = 400000, kBlkMinBoth = 300000;
constexpr int64_t kBlkMinGather = 2000000;
constexpr int64_t kNodeMaxSpread = 400000;
// FP64 with gathers: blocks from 400 k points (with interpolation on 0.6 M leaves
// 205 us, 238 by ranges, 208 by tiles; 1 M 294, 478, 354) or where four to a leaf
// are there (400 k on 14 k leaves 204, 236, 287), ranges below that (200 k on 2.7 M
// leaves 215 by ranges, 392 by tiles; markers there 197 and 150).
constexpr int64_t kBlkMinF64Both = 400000, kBlkMinF64Crowded = 250000, kNodeMaxF64Both = 250000;
// Plans that do not spread have only the sharing of lookups and field rows to
// gain, so their line also asks for leaves that caches do not hold, or for more
// points; and a root of more than one cube, since a sort by one block has one
// digit.  Interpolation, FP32, tiles of points sorted by host against block
// pass: 4 M random points on 14 k leaves 261 and 321 us, 38 k 273 and 283, 0.6 M 366
// and 293, 2.7 M 449 and 322; 10^7 on 14 k 705 and 733 (markers 853 and 581), 38 k
// 736 and 657, on 512 leaves, one cube, 643 and 1907; 2 M on 4,096 leaves without
// sub-tables 146 and 143.  With both outputs blocks gain less (14 k leaves, 10^7
// points, 1020 and 1146).
constexpr int64_t kBlkMinGatherLeaves = 131072, kBlkMinGatherFew = 8000000;
// FP32 atomic sums in FP64 (blocks and ranges) cost 60 bytes a leaf and a launch
// where FP32 ones cost 12: 10 us a million leaves, 0.18 ms of 17 M.  On larger
// trees than this plans keep to tiles of points sorted by host and FP32 sums (100 k
// points on 17 M leaves 317 us wide, 230 by tiles; 4 M 1574 and 1042), and plain
// calls do not sort fewer points than a 64th of the leaves (100 k points in
// host order 154 unsorted, 320 wide; 300 k 737 and 406, random ones 1152 and 408).
constexpr int64_t kWideMaxLeaves = 4000000;
static bool wide_fits(const ot_tree *t, int64_t n, bool plan)
{
    return t->n_leaves <= kWideMaxLeaves || (plan ? 2 : 64) * n >= t->n_leaves;
}

SortedRoute sorted_route(const ot_tree *t, int64_t n, int ops, int dtype, int mode, bool plan)
{
    SortedRoute r{false, false, false};
    const bool spread = (ops & kOpSpread) != 0, gathers = (ops & (kOpInterp | kOpGrad)) != 0;
    const bool f32_sums = spread && dtype == OT_F32 && mode == OT_SPREAD_ATOMIC;
    const bool blocks = t->view.lev[0] >= kBlkBits && n >= 64 * (int64_t)t->view.nblk && n < (int64_t(1) << 31);
    if (!(ops & ~kOpLocate) || (f32_sums && !wide_fits(t, n, plan))) return r;
    if (!spread) {
        const bool one_output = !(ops & kOpInterp) || !(ops & kOpGrad);
        r.blocks = blocks && n >= kBlkMinGather &&
                   (t->n_leaves >= kBlkMinGatherLeaves ||
                    (one_output && t->view.lev[0] > kBlkBits &&
                     (t->view.nblk == t->view.blk1 || n >= kBlkMinGatherFew)));
        return r;
    }
    const bool dense = 3 * n >= t->n_leaves;
    if (dtype == OT_F64 && gathers) {
        r.blocks = blocks && ((dense && n >= kBlkMinF64Both) || (n >= kBlkMinF64Crowded && n >= 4 * t->n_leaves));
        r.nodes = !r.blocks && (n < kNodeMaxF64Both || 32 * n < t->n_leaves);
    } else {
        r.blocks = blocks && dense && n >= (gathers ? kBlkMinBoth : kBlkMinSpread);
        r.nodes = !r.blocks && (n < kNodeMaxSpread || 16 * n < t->n_leaves || (f32_sums && !plan));
    }
    r.wide = f32_sums && (r.blocks || r.nodes);
    return r;
}

// Which plain calls that search the hosts themselves are sorted (track.hip).
bool plain_sorts(const ot_tree *t, int64_t n, int ops, int dtype, int mode)
{
    const bool f32_sums = dtype == OT_F32 && mode == OT_SPREAD_ATOMIC;
    const bool f64_gathers = dtype == OT_F64 && (ops & (kOpInterp | kOpGrad));
    const int64_t least = f32_sums ? kSortMinF32Sums : f64_gathers ? kSortMinF64Both : kSortMinSpread;
    return (ops & kOpSpread) && t->n_leaves > kFewLeaves && n >= least && n <= INT32_MAX &&
           (!f32_sums || wide_fits(t, n, false));
}

// Sorted plans of so few points that the plain passes are faster unsorted
// (30 k points on 38 k leaves: spreading 51 against 61 us, interpolation 10
// against 47; 100 k: spreading 66 sorted against 134, interpolation 16; on 512
// leaves at any size, 390 k points 71 against 219).  Not for atomic spreading:
// an unsorted pass adds to a leaf more often, and the sums were up to 3 times
// less exact (FP64, 50 k random points on 4,096 leaves 3.5e-16 -> 6.4e-16, on 512
// leaves 4.3e-16 -> 1.3e-15).  FP64 sums of up to 1,024 points, in 37 workgroups
// of 28, are as exact as those of 16 tiles of 64 (13 us against 30).
constexpr int64_t kSmallAtomic = 1024;
bool small_rule(const ot_tree *t, int64_t n, int ops, int dtype, int mode)
{
    if (n <= 0 || !(ops & ~kOpLocate)) return false;
    if (!(ops & kOpSpread)) return n < 100000;
    const bool atomic = mode == OT_SPREAD_ATOMIC;
    if (t->n_leaves <= kFewLeaves) return !atomic;
    return atomic ? dtype == OT_F64 && n <= kSmallAtomic : n < kSortMinSpread;
}

}  // namespace ot
