// Block pass of sorted plans: one workgroup takes the points of one block of
// host cells and works on a dense grid of the block's stencil nodes in LDS.
//
// A block is a cube of 8^3 root cells (its hosts are the root-level leaves in
// it) or one sub-table of the descent table (its hosts are the leaves below
// one split cell, up to three levels deeper).  The points arrive sorted by
// block (point_sort.hip).  For each level l of a block's hosts the stencil
// nodes are the level-l cells of the block and one cell around it, a grid of
// (2^g + 2)^3 nodes for a block of 2^g cells a side (10^3, 6^3 and 4^3).
// Every node's leaf is looked up once per tile of points, its field value is
// loaded to LDS once, and its spreading sum is kept in LDS until the tile
// ends; a point finds its 27 nodes at fixed offsets from its host's node, so
// the per-point work has no table lookups, no hashing and no gathers from
// device memory.
//
// A tile's points are ordered by host (a counting sort of 16-bit indices in
// LDS) and taken in chunks of one point per thread.  Each thread interpolates
// its point from the LDS grid and leaves the point's weights and force in
// LDS; then groups of three lanes take runs of up to kRun points of one host,
// one plane of nodes each: the 27 sums of a lane stay in registers over the
// run, so the spreading's LDS adds are one per run and node component instead
// of one per point and node component (LDS atomics run at a few lanes per
// clock on this target and had bounded the per-point pass).
//
// Measured (FP32, fixed point, interpolation and spreading): 10^7 points on a
// tree of 2.66 M leaves 0.60 ms against 1.05 of the per-point pass, 10^8 points
// in shells on 20 M leaves 5.8 against 10.7 ms; the sort passes need the block
// bits only (two passes instead of three above 4 M leaves).
//
// Values are those of the per-point pass: the same weights, the same order of
// the interpolation sums and the same rounded fixed-point contributions.
// Blocks with few points are left to short ranges of points (node_pass.h): a
// tile's grid costs more than their points do.
#pragma once

#include <hip/hip_runtime.h>

#include "batch_plan.h"
#include "ot_common.h"
#include "track_device.h"

namespace ot {

// Points [start, start + count) of block `key`: a cell at level l0 with
// coordinates a there, whose hosts are at levels l0 + 1 .. l0 + d (root cubes:
// l0 + d).
struct BlkTile {
    uint32_t start, count, key;
    int32_t l0;
    uint32_t a[3];
    int32_t d;
};

// Device words of a plan's block pass, zeroed before each run: counts of
// tiles and ranges, and the tile queues.
enum : int { kBlkRootTiles = 3, kBlkSubTiles = 4, kBlkRanges = 5, kBlkRootQueue = 6, kBlkSubQueue = 7 };
constexpr int kBlkWindow = 256;     // most points per range of points in sparse blocks
// Fewest points of a block that gets tiles: a tile's grid (lookups, field
// loads, clears, flush) costs about as much as the other passes over a few
// hundred points.  Measured on 16.9 M points in 17.1 M leaves (60 k sub-tables
// of ~37 points): from 192 points 1.04 ms (sparse blocks) + 0.01 (tiles), from 64
// points 0.95 + 0.81, from 24 points 0.80 + 1.37.
constexpr int kBlkDense = 192;
constexpr int kBlkTilePts = 3072;   // most points per tile
constexpr int kBlkTileMin = 768;    // least points a block's tiles are cut down to
constexpr int kRun = 6;             // most points per run (8: +3% on shells, 4: +1 to 2%)

// Nodes of a block's grids: the 10^3 grid first, then (sub-tables) 6^3 and 4^3.
template <bool ROOT>
struct BlkGrid {
    static constexpr int kNodes = ROOT ? 1000 : 1280;
};

__device__ __forceinline__ int blk_off(int g) { return g == 3 ? 0 : (g == 2 ? 1000 : 1216); }
__device__ __forceinline__ int blk_edge(int g) { return (1 << g) + 2; }

constexpr uint32_t kBlkNoNode = 0xFFFFFFFFu;   // a node beyond a wall, or of a grid the block does not have

// Threads of a workgroup.  Root cubes: two workgroups of 512 per CU (FP32; one
// of 1024 was 13% slower).  Sub-tables: one of 768 (two of 384 took 7.35 ms in
// shells of 10^8 points against 5.74: the grids and lookups of a tile then
// serve twice the threads, and the tiles in flight fit an XCD's L2, where the
// points are read a second time in host order; 512 and 1024 took 6.4 and 6.0).
// FP64: one workgroup either way, 512 threads to keep 256 registers.
template <typename T, bool ROOT>
struct BlkThreads {
    static constexpr int value = (ROOT || sizeof(T) == 8) ? 512 : 768;
    static constexpr int waves = sizeof(T) == 8 ? 2 : (ROOT ? 4 : 3);   // per SIMD
};

template <typename T, int MODE, int OPS, bool ROOT>
struct BlkShared {
    using Acc = typename AccType<T, MODE>::type;
    static constexpr int NN = BlkGrid<ROOT>::kNodes;
    static constexpr int NT = BlkThreads<T, ROOT>::value;
    static constexpr bool kGather = (OPS & (kOpInterp | kOpGrad)) != 0;
    static constexpr bool kSpread = (OPS & kOpSpread) != 0;
    uint32_t ent[NN];
    T u[kGather ? 3 : 1][kGather ? NN : 1];
    Acc acc[kSpread ? NN : 1][3];
    // per sorted point of the chunk: (w_x[3], F_x), (w_y[3], F_y), (w_z[3], F_z)
    T rec[kSpread ? NT : 1][12];
    uint32_t bins[NN / 2 + 1];        // host counts, then the hosts' first sorted positions, 16 bits each
    uint16_t perm[kBlkTilePts];       // sorted position -> point of the tile
    uint32_t runs[kSpread ? NT : 1];  // first point | host node << 10 | (points - 1) << 21
    uint32_t rcnt[kRun], rcur[kRun];
    uint32_t wsum[NT / 64];
    unsigned next;                    // the tile after this one
    BlkTile tile;
};

// Level-l cell of coordinate x along one axis (wrapped when periodic; hosted
// points of walled domains lie inside), exact as point_cell's.
template <typename T>
__device__ __forceinline__ int blk_cell(T x, int l, int periodic)
{
    const T sc = (T)(1 << l);
    T f = floor(x * sc);
    if (periodic) f -= floor(f * ldexp(T(1), -l)) * sc;
    return (int)f;
}

// One point's result at its input row.  stream: an output larger than the
// memory-side cache, whose scattered rows only push other lines out (measured
// in shells of 10^8 points: 7.9 -> 7.4 ms; on 10^7 points 0.58 -> 0.64, not taken).
template <typename T>
__device__ __forceinline__ void blk_store(T *p, const T (&v)[3], bool stream)
{
    if (stream) {
#pragma unroll
        for (int c = 0; c < 3; ++c) __builtin_nontemporal_store(v[c], p + c);
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) p[c] = v[c];
    }
}
constexpr int64_t kBlkStreamBytes = int64_t(256) << 20;

// The node that stands for the leaf of node q (grid g, cell n at level
// l0 + g) when the leaf is coarser than the grid: the leaf's cell in the grid
// of its own level, or of its cells in the coarsest grid the first one there.
// All of a leaf's nodes then reach device memory with one add, as one table
// slot of the per-point pass would (atomic sums are rounded there).
__device__ __forceinline__ int blk_canonical(int level, int l0, const uint32_t a[3], int g, const int n[3])
{
    const int gg = max(level - l0, 1), k = max(l0 + 1 - level, 0);
    int q = blk_off(gg), s = 1;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int lo = (int)(a[c] << gg) - 1;
        const int m = ((n[c] >> (g - gg)) >> k) << k;
        q += s * (max(m, lo) - lo);
        s *= blk_edge(gg);
    }
    return q;
}

// Grid, and coordinates inside it, of node q.
template <bool ROOT>
__device__ __forceinline__ int blk_node(int q, int x[3])
{
    if (ROOT || q < 1000) {
        x[0] = q % 10;
        x[1] = (q / 10) % 10;
        x[2] = q / 100;
        return 3;
    }
    if (q < 1216) {
        q -= 1000;
        x[0] = q % 6;
        x[1] = (q / 6) % 6;
        x[2] = q / 36;
        return 2;
    }
    q -= 1216;
    x[0] = q & 3;
    x[1] = (q >> 2) & 3;
    x[2] = q >> 4;
    return 1;
}

template <typename T, int MODE, int OPS, bool ROOT>
__global__ __launch_bounds__((BlkThreads<T, ROOT>::value), (BlkThreads<T, ROOT>::waves)) void k_block(
    TreeView tv, const BlkTile *__restrict__ tiles, const unsigned *__restrict__ n_tiles, unsigned *__restrict__ queue,
    const uint64_t *__restrict__ kv, const T *__restrict__ rec, const T *__restrict__ field, T *__restrict__ vel,
    T *__restrict__ fout, unsigned long long *__restrict__ facc, FxRef fx, T *__restrict__ grad, bool stream)
{
    using Sh = BlkShared<T, MODE, OPS, ROOT>;
    using Acc = typename Sh::Acc;
    constexpr int NN = Sh::NN, NT = Sh::NT;
    constexpr int RS = (OPS & (kOpSpread | kOpGrad)) ? 6 : 3;
    constexpr int kPer = kBlkTilePts / NT;
    static_assert(kBlkTilePts % NT == 0 && NT <= 1024 && NN <= 2048 && kRun <= 8, "packing of runs");
    __shared__ Sh sh;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const double scale = (Sh::kSpread && MODE == kModeFixed) ? fx_scale<T>(fx) : 1.0;
    const unsigned nt = *n_tiles;
    const int rsh = tv.L - tv.lev[0];
    if (nt == 0u) return;
    if (tid == 0) {
        sh.next = atomicAdd(queue, 1u);
        if (sh.next < nt) sh.tile = tiles[sh.next];
    }
    __syncthreads();

    for (;;) {
        if (sh.next >= nt) break;   // uniform
        const BlkTile tile = sh.tile;
        const int cnt = (int)tile.count;
        const int l0 = ROOT ? tv.lev[0] - kBlkBits : tile.l0, d = ROOT ? kBlkBits : tile.d;
        const uint32_t a[3] = {tile.a[0], tile.a[1], tile.a[2]};
        const T *trec = rec + (int64_t)RS * tile.start;
        const uint64_t *tkv = kv + tile.start;
        // the next tile is claimed now and its description loaded before the
        // flush, so neither is waited for
        unsigned nxt = 0u;
        if (tid == 0) nxt = atomicAdd(queue, 1u);

        // ---- the points' positions (and host levels), and the nodes' root
        // entries, all in flight together; sums and host counts cleared
        T X[kPer][3];
        uint32_t hi[ROOT ? 1 : kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = j * NT + tid < cnt ? j * NT + tid : 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) X[j][c] = trec[RS * i + c];
            if (!ROOT) hi[j] = reinterpret_cast<const uint32_t *>(tkv)[2 * i + 1];
        }
        constexpr int kN = (NN + NT - 1) / NT;
        uint32_t e[kN], N[kN][3];
        bool in[kN];
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            const int q = j * NT + tid;
            int x[3];
            const int g = blk_node<ROOT>(q, x);
            const int l = l0 + g, s = tv.L - l;
            const int32_t M = 1 << l;
            in[j] = q < NN && (ROOT || g <= d);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                int32_t n = (int32_t)(a[c] << g) + x[c] - 1;
                if (tv.periodic) n &= M - 1;
                else in[j] = in[j] && n >= 0 && n < M;
                N[j][c] = in[j] ? ((uint32_t)n << s) | (s > 0 ? 1u << (s - 1) : 0u) : 0u;
            }
            e[j] = ld_table(tv, in[j] ? interleave3(N[j][0] >> rsh, N[j][1] >> rsh, N[j][2] >> rsh) : 0u);
        }
        if constexpr (Sh::kSpread) {
            Acc *z = &sh.acc[0][0];
            for (int i = tid; i < 3 * NN; i += NT) z[i] = Acc(0);
            if (tid < kRun) {
                sh.rcnt[tid] = 0u;
                sh.rcur[tid] = 0u;
            }
        }
        for (int i = tid; i < NN / 2 + 1; i += NT) sh.bins[i] = 0u;
        __syncthreads();

        // ---- counting sort of the tile's points by host: host counts
        uint32_t hr[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (j * NT >= cnt) break;   // uniform
            const int g = ROOT ? kBlkBits : (int)((hi[j] >> kLevelShift) & 31u) - l0;
            const int E = ROOT ? 10 : blk_edge(g);
            int h = ROOT ? 0 : blk_off(g), s = 1;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                h += s * (blk_cell<T>(X[j][c], l0 + g, tv.periodic) - (int)(a[c] << g) + 1);
                s *= E;
            }
            if (j * NT + tid < cnt) {
                const int sft = 16 * (h & 1);
                hr[j] = (uint32_t)h << 16 | ((atomicAdd(&sh.bins[h >> 1], 1u << sft) >> sft) & 0xFFFFu);
            }
        }
        // the nodes' level-1 entries and deeper, then their field rows (in
        // flight during the rest of the sort)
        uint32_t e1[kN];
#pragma unroll
        for (int j = 0; j < kN; ++j) e1[j] = ld_table(tv, step1_index(tv, e[j], N[j][0], N[j][1], N[j][2]));
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            if (e[j] & kSplit) e[j] = e1[j];
            if (e[j] & kSplit) e[j] = descend_from_level2(tv, e[j], N[j][0], N[j][1], N[j][2]);
        }
        T f[Sh::kGather ? kN : 1][3];
        if constexpr (Sh::kGather) {
#pragma unroll
            for (int j = 0; j < kN; ++j) {
                const int64_t i = 3 * (int64_t)(in[j] ? e[j] & kIdMask : 0u);
#pragma unroll
                for (int c = 0; c < 3; ++c) f[j][c] = field[i + c];
            }
        }
        __syncthreads();
        {
            // exclusive prefix of the counts, in place
            constexpr int kW = (NN / 2 + NT - 1) / NT;   // packed words per thread
            uint32_t v[kW], sum = 0u;
#pragma unroll
            for (int w = 0; w < kW; ++w) {
                const int i = tid * kW + w;
                v[w] = i < NN / 2 ? sh.bins[i] : 0u;
                sum += (v[w] & 0xFFFFu) + (v[w] >> 16);
            }
            uint32_t x = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (lane == 63) sh.wsum[wid] = x;
            __syncthreads();
            uint32_t pre = x - sum;
#pragma unroll
            for (int w = 0; w < NT / 64; ++w) pre += w < wid ? sh.wsum[w] : 0u;
#pragma unroll
            for (int w = 0; w < kW; ++w) {
                const int i = tid * kW + w;
                const uint32_t lo = v[w] & 0xFFFFu;
                if (i < NN / 2) sh.bins[i] = pre | (pre + lo) << 16;
                pre += lo + (v[w] >> 16);
            }
            if (tid == NT - 1) sh.bins[NN / 2] = (uint32_t)cnt;
            __syncthreads();
        }
        const uint16_t *first = reinterpret_cast<const uint16_t *>(sh.bins);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (j * NT >= cnt) break;
            if (j * NT + tid < cnt) sh.perm[first[hr[j] >> 16] + (hr[j] & 0xFFFFu)] = (uint16_t)(j * NT + tid);
        }
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            const int q = j * NT + tid;
            if (q < NN) {
                sh.ent[q] = in[j] ? e[j] : kBlkNoNode;
                if constexpr (Sh::kGather) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) sh.u[c][q] = in[j] ? f[j][c] : T(0);
                }
            }
        }
        __syncthreads();

        // ---- chunks of NT sorted points.  (Loading a chunk's records during
        // the one before it cost registers that spilled: 529 -> 574 us.)
        for (int c0 = 0; c0 < cnt; c0 += NT) {
            const int i = c0 + tid;
            const int cend = min(c0 + NT, cnt);
            int rl = 0, h = 0;   // this thread's run (0: none starts here)
            if (i < cnt) {
                const int k = sh.perm[i];
                const T Y[3] = {trec[RS * k], trec[RS * k + 1], trec[RS * k + 2]};
                T F[3] = {T(0), T(0), T(0)};
                if (RS == 6) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[c] = trec[RS * k + 3 + c];
                }
                const uint64_t wd = tkv[k];
                const int64_t kd = (int64_t)(uint32_t)wd;
                const int g = ROOT ? kBlkBits : (int)((uint32_t)(wd >> 58) & 31u) - l0;
                const int E = ROOT ? 10 : blk_edge(g), l = l0 + g;
                const T sc = (T)(1 << l);
                T w[3][3], dw[3][3];
                h = ROOT ? 0 : blk_off(g);
                int s = 1;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    h += s * (blk_cell<T>(Y[c], l, tv.periodic) - (int)(a[c] << g) + 1);
                    s *= E;
                    T t, r;
                    cell_offsets<T>(Y[c] * sc, t, r);
                    delta3<T>(t, r, w[c]);
                    if (OPS & kOpGrad) {
                        T wt[3];
                        delta3_grad<T>(t, r, wt, dw[c]);
#pragma unroll
                        for (int o = 0; o < 3; ++o) dw[c][o] *= sc;
                    }
                }
                if constexpr (Sh::kSpread) {
                    T *rw = sh.rec[tid];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
#pragma unroll
                        for (int o = 0; o < 3; ++o) rw[4 * c + o] = w[c][o];
                        rw[4 * c + 3] = F[c];
                    }
                    const int b = max((int)first[h], c0), z = min((int)first[h + 1], cend);
                    if ((i - b) % kRun == 0) {
                        rl = min(kRun, z - i);
                        atomicAdd(&sh.rcnt[rl - 1], 1u);
                    }
                }
                if constexpr (Sh::kGather) {
                    T U[3] = {T(0), T(0), T(0)}, G[3] = {T(0), T(0), T(0)};
#pragma unroll
                    for (int oz = 0; oz < 3; ++oz) {
#pragma unroll
                        for (int oy = 0; oy < 3; ++oy) {
                            const int q = h - 1 + E * ((oy - 1) + E * (oz - 1));
#pragma unroll
                            for (int ox = 0; ox < 3; ++ox) {
                                const T f0 = sh.u[0][q + ox], f1 = sh.u[1][q + ox], f2 = sh.u[2][q + ox];
                                if (OPS & kOpInterp) {
                                    const T ww = w[0][ox] * w[1][oy] * w[2][oz];
                                    U[0] = fma(ww, f0, U[0]);
                                    U[1] = fma(ww, f1, U[1]);
                                    U[2] = fma(ww, f2, U[2]);
                                }
                                if (OPS & kOpGrad) {
                                    const T dot = fma(F[0], f0, fma(F[1], f1, F[2] * f2));
                                    G[0] = fma(dot * dw[0][ox], w[1][oy] * w[2][oz], G[0]);
                                    G[1] = fma(dot * w[0][ox], dw[1][oy] * w[2][oz], G[1]);
                                    G[2] = fma(dot * w[0][ox], w[1][oy] * dw[2][oz], G[2]);
                                }
                            }
                        }
                    }
                    if (OPS & kOpInterp) blk_store(vel + 3 * kd, U, stream);
                    if (OPS & kOpGrad) blk_store(grad + 3 * kd, G, stream);
                }
            }
            if constexpr (Sh::kSpread) {
                __syncthreads();
                // runs ordered by length, the longest first, so that the
                // lanes of a wave stop together
                uint32_t nruns = 0u, at = 0u;
#pragma unroll
                for (int r = kRun - 1; r >= 0; --r) {
                    if (rl - 1 == r) at = nruns;
                    nruns += sh.rcnt[r];
                }
                if (rl) {
                    at += atomicAdd(&sh.rcur[rl - 1], 1u);
                    sh.runs[at] = (uint32_t)tid | (uint32_t)h << 10 | (uint32_t)(rl - 1) << 21;
                }
                __syncthreads();
                if (tid < kRun) {   // for the next chunk
                    sh.rcnt[tid] = 0u;
                    sh.rcur[tid] = 0u;
                }
                const int grp = lane / 3, oz = lane - 3 * grp;
                for (uint32_t j0 = (uint32_t)wid * 21u; j0 < nruns; j0 += (NT / 64) * 21u) {
                    const uint32_t j = j0 + (uint32_t)grp;
                    if (grp < 21 && j < nruns) {
                        const uint32_t rw = sh.runs[j];
                        const int p0 = (int)(rw & 1023u), hn = (int)((rw >> 10) & 2047u), m = (int)(rw >> 21) + 1;
                        Acc s[9][3];
#pragma unroll
                        for (int q = 0; q < 9; ++q) s[q][0] = s[q][1] = s[q][2] = Acc(0);
                        for (int p = 0; p < m; ++p) {
                            const T *r = sh.rec[p0 + p];
                            const T wz = r[8 + oz];
                            const double F0 = (double)r[3] * scale, F1 = (double)r[7] * scale, F2 = (double)r[11] * scale;
#pragma unroll
                            for (int q = 0; q < 9; ++q) {
                                const double ww = (double)(r[q % 3] * r[4 + q / 3] * wz);
                                if constexpr (MODE == kModeFixed) {
                                    s[q][0] += (unsigned long long)__double_as_longlong(fma(ww, F0, kFxMagic));
                                    s[q][1] += (unsigned long long)__double_as_longlong(fma(ww, F1, kFxMagic));
                                    s[q][2] += (unsigned long long)__double_as_longlong(fma(ww, F2, kFxMagic));
                                } else {
                                    s[q][0] = fma(ww, F0, s[q][0]);
                                    s[q][1] = fma(ww, F1, s[q][1]);
                                    s[q][2] = fma(ww, F2, s[q][2]);
                                }
                            }
                        }
                        const int E = ROOT ? 10 : (hn < 1000 ? 10 : (hn < 1216 ? 6 : 4));
                        // the magic number's bits, once per point of the run
                        const unsigned long long mb = (unsigned long long)m * kFxMagicBits;
#pragma unroll
                        for (int q = 0; q < 9; ++q) {
                            const int nd = hn - 1 + q % 3 + E * ((q / 3 - 1) + E * (oz - 1));
#pragma unroll
                            for (int c = 0; c < 3; ++c) {
                                if constexpr (MODE == kModeFixed) atomicAdd(&sh.acc[nd][c], s[q][c] - mb);
                                else atomicAdd(&sh.acc[nd][c], s[q][c]);
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
        BlkTile nd;
        if (tid == 0 && nxt < nt) nd = tiles[nxt];

        // ---- the nodes' sums to device memory, neighbouring lanes on one
        // node's three components
        if constexpr (Sh::kSpread) {
            if (!ROOT) {
                // nodes of leaves coarser than their grid add to one of them
                for (int q = tid; q < NN; q += NT) {
                    int x[3];
                    const int g = blk_node<ROOT>(q, x);
                    const uint32_t en = sh.ent[q];
                    const int lv = (int)((en >> kLevelShift) & 31u);
                    if (g > d || en == kBlkNoNode || lv >= l0 + g) continue;
                    int n[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) n[c] = (int)(a[c] << g) + x[c] - 1;
                    const int to = blk_canonical(lv, l0, a, g, n);
                    if (to == q) continue;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const Acc v = sh.acc[q][c];
                        if (v != Acc(0)) {
                            atomicAdd(&sh.acc[to][c], v);
                            sh.acc[q][c] = Acc(0);
                        }
                    }
                }
                __syncthreads();
            }
            for (int i = tid; i < 3 * NN; i += NT) {
                const int q = i / 3, c = i - 3 * q;
                const Acc v = sh.acc[q][c];
                const uint32_t en = sh.ent[q];
                if (v != Acc(0) && en != kBlkNoNode) global_add<T, MODE>(fout, facc, 3 * (int64_t)(en & kIdMask) + c, v);
            }
        }
        if (tid == 0) {
            sh.next = nxt;
            if (nxt < nt) sh.tile = nd;
        }
        __syncthreads();   // the next tile reuses everything
    }
}

// Finds the blocks among the sorted words and lists the passes' work (block.hip).
void enqueue_bounds(const ot_tree *t, BlkWork &w, const uint64_t *kv, hipStream_t s);

}  // namespace ot
