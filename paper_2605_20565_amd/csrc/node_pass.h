// Node-parallel passes: nine lanes per point, each with one x-row of three
// stencil nodes.  k_nodes takes small plain calls, k_node_ranges ranges of
// sorted points that are too few or too sparse for the other passes.
//
// A small call's time is latency: with one thread per point a wave walks a
// straight line of ~5,000 instructions (27 unrolled nodes) whose code it
// fetches cold, with few waves on the chip to overlap it.  Here a point's
// nodes are looked up, gathered and spread side by side, in a short loop-free
// kernel with nine times the lanes.  Values are those of the per-point pass:
// the interpolation's 27 products go through LDS to one lane per component,
// which sums them in the same order; spreading goes through the same LDS table
// (leaf-keyed, one device add per slot), so atomic FP32 sums keep their FP64
// partial sums.  Spreading random points is then bound by the device's atomic
// units: about 26 lines a point at 21 G line operations per second.  The sizes
// it is chosen for, and both sides' times, are in track.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "ot_common.h"
#include "track_device.h"

namespace ot {

constexpr int kNodeLanes = 9;                                        // lanes per point: (oy, oz)
constexpr int kNodeWavePts = 64 / kNodeLanes;                        // 7; lane 63 idles
constexpr int kNodeThreads = 256;
constexpr int kNodePts = kNodeWavePts * (kNodeThreads / 64);         // 28 points per workgroup
constexpr int kNodeSlots = 1024;                                     // spreading table (28 x 27 nodes at most)
// Sorted ranges: one table for all points of a range.
constexpr int kRangeThreads = 512;
constexpr int kRangePts = kNodeWavePts * (kRangeThreads / 64);       // points per step
constexpr int kRangeSlots = 2048;

// Values per node in LDS: weight and field row; gradient alone: two factors
// per node and three per row of three nodes (81 a point).  With these, two
// workgroups of k_node_ranges share a CU's LDS in every FP32 variant; six
// values per node left room for one.
template <int OPS>
struct NodeVals { static constexpr int value = (OPS & kOpInterp) ? 4 : 3; };

// This lane's place: point of the wave, row of nodes, point of the workgroup.
struct NodeLane {
    int p, row, oy, oz, slot;
    bool used;
    __device__ __forceinline__ NodeLane()
    {
        const int lane = threadIdx.x & 63;
        p = lane / kNodeLanes;
        row = lane - kNodeLanes * p;
        oy = row % 3;
        oz = row / 3;
        used = p < kNodeWavePts;
        slot = (int)(threadIdx.x >> 6) * kNodeWavePts + (used ? p : 0);
    }
};

// A lane's three nodes: leaf entry, root cell, and whether the node exists.
struct NodeRow {
    uint32_t ent[3], root[3];
    bool in[3];
};

// The leaves of this lane's row of nodes of the cell I at its host level l.
template <bool PER>
__device__ __forceinline__ void node_row(const TreeView &tv, const NodeLane &ln, const uint32_t (&I)[3], int l, bool ok,
                                         NodeRow &nr)
{
    const int sh = tv.L - l, rsh = tv.L - tv.lev[0];
    const int32_t M = 1 << l;
    const uint32_t half = sh > 0 ? 1u << (sh - 1) : 0u;
    uint32_t N[3][3], sub[3];
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) {
        const int o[3] = {ox, ln.oy, ln.oz};
        nr.in[ox] = ok;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int32_t c = (int32_t)(I[d] >> sh) + o[d] - 1;
            if (PER) c &= M - 1;
            else nr.in[ox] = nr.in[ox] && c >= 0 && c < M;
            N[ox][d] = ((uint32_t)c << sh) | half;
        }
        if (!nr.in[ox]) N[ox][0] = N[ox][1] = N[ox][2] = 0u;
        nr.root[ox] = interleave3(N[ox][0] >> rsh, N[ox][1] >> rsh, N[ox][2] >> rsh);
        nr.ent[ox] = ld_table(tv, nr.root[ox]);
    }
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) sub[ox] = ld_table(tv, step1_index(tv, nr.ent[ox], N[ox][0], N[ox][1], N[ox][2]));
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) {
        if (nr.ent[ox] & kSplit) nr.ent[ox] = sub[ox];
        if (nr.ent[ox] & kSplit) nr.ent[ox] = descend_from_level2(tv, nr.ent[ox], N[ox][0], N[ox][1], N[ox][2]);
    }
}

// One point per nine lanes, all threads of the workgroup: position X, host
// entry e (ok: it has one), force F; results to index kd (have: there is a
// point).  buf: LDS, one entry per point of the workgroup.
template <typename T, int OPS, int MODE, bool PER, int S>
__device__ __forceinline__ void node_step(const TreeView &tv, const NodeLane &ln, const T (&X)[3], const uint32_t (&I)[3],
                                          uint32_t e, bool ok, bool have, const T (&F)[3], int64_t kd,
                                          const T *__restrict__ field, T *__restrict__ vel, T *__restrict__ grad,
                                          LdsSink<T, MODE, S> &sink, T (*buf)[27][NodeVals<OPS>::value])
{
    constexpr bool kInterp = (OPS & kOpInterp) != 0, kGrad = (OPS & kOpGrad) != 0, kSpread = (OPS & kOpSpread) != 0;
    constexpr bool kGather = kInterp || kGrad;
    using Acc = typename AccType<T, MODE>::type;
    const int row = ln.row, oy = ln.oy, oz = ln.oz, slot = ln.slot;
    // the stencil's 1-D weights, and this lane's three nodes
    const int l = (int)((e >> kLevelShift) & 31u);
    const T sc = (T)(1 << l);
    T w[3][3], dw[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T t, r;
        cell_offsets<T>(X[d] * sc, t, r);
        delta3<T>(t, r, w[d]);
        if (kGrad) {
            T wt[3];
            delta3_grad<T>(t, r, wt, dw[d]);
#pragma unroll
            for (int o = 0; o < 3; ++o) dw[d][o] *= sc;
        }
    }
    NodeRow nr;
    node_row<PER>(tv, ln, I, l, ok, nr);
    const uint32_t (&ent)[3] = nr.ent, (&root)[3] = nr.root;
    const bool (&in)[3] = nr.in;
    // a lane's own row of weights, picked without indexing registers by lane
    const T wy = oy == 0 ? w[1][0] : oy == 1 ? w[1][1] : w[1][2];
    const T wz = oz == 0 ? w[2][0] : oz == 1 ? w[2][1] : w[2][2];

    if constexpr (kGather) {
        T f[3][3];
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
            const int64_t j = 3 * (int64_t)(in[ox] ? ent[ox] & kIdMask : 0u);
#pragma unroll
            for (int c = 0; c < 3; ++c) f[ox][c] = field[j + c];
        }
        if constexpr (kInterp) {
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                T *b = buf[slot][3 * row + ox];
                if (ln.used) {
                    b[0] = w[0][ox] * wy * wz;
#pragma unroll
                    for (int c = 0; c < 3; ++c) b[1 + c] = in[ox] ? f[ox][c] : T(0);
                }
            }
            __syncthreads();
            if (row < 3 && have) {
                T U = T(0);
#pragma unroll
                for (int q = 0; q < 27; ++q) U = fma(buf[slot][q][0], buf[slot][q][1 + row], U);
                vel[3 * kd + row] = ok ? U : T(0);
            }
            if (kGrad) __syncthreads();
        }
        if constexpr (kGrad) {
            T *g = &buf[slot][0][0];
            const T dy = oy == 0 ? dw[1][0] : oy == 1 ? dw[1][1] : dw[1][2];
            const T dz = oz == 0 ? dw[2][0] : oz == 1 ? dw[2][1] : dw[2][2];
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const T dot = fma(F[0], f[ox][0], fma(F[1], f[ox][1], F[2] * f[ox][2]));
                if (ln.used) {
                    g[2 * (3 * row + ox)] = in[ox] ? dot * dw[0][ox] : T(0);
                    g[2 * (3 * row + ox) + 1] = in[ox] ? dot * w[0][ox] : T(0);
                }
            }
            if (ln.used) {
                g[54 + 3 * row] = wy * wz;
                g[54 + 3 * row + 1] = dy * wz;
                g[54 + 3 * row + 2] = wy * dz;
            }
            __syncthreads();
            if (row < 3 && have) {
                T G = T(0);
#pragma unroll
                for (int q = 0; q < 27; ++q) G = fma(g[2 * q + (row > 0)], g[54 + 3 * (q / 3) + row], G);
                grad[3 * kd + row] = ok ? G : T(0);
            }
        }
    }
    if constexpr (kSpread) {
        uint32_t at[3];
        bool hit[3];
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
            hit[ox] = false;
            at[ox] = 0u;
            if (in[ox]) {
                const uint32_t leaf = ent[ox] & kIdMask;
                at[ox] = sink.primary(ent[ox], root[ox], tv.lev[0]);
                const uint32_t old = atomicCAS(&sink.keys[at[ox]], 0u, leaf + 1u);
                hit[ox] = old == 0u || old == leaf + 1u;
            }
        }
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
            if (!in[ox]) continue;
            const T ww = w[0][ox] * wy * wz;
            Acc a[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c] = to_acc<T, MODE>(ww, F[c], sink.scale);
            if (hit[ox]) {
#pragma unroll
                for (int c = 0; c < 3; ++c) atomicAdd(&sink.vals[3 * at[ox] + c], a[c]);
            } else {
                sink.add_probing(ent[ox] & kIdMask, at[ox], a[0], a[1], a[2]);
            }
        }
    }
}

template <typename T, int OPS, int MODE, bool PER>
__global__ __launch_bounds__(kNodeThreads) void k_nodes(TreeView tv, int64_t n, const T *__restrict__ pos,
                                                        const T *__restrict__ field, const T *__restrict__ force,
                                                        int32_t *__restrict__ ids, T *__restrict__ vel,
                                                        T *__restrict__ fout, unsigned long long *__restrict__ facc,
                                                        FxRef fx, T *__restrict__ grad,
                                                        const int32_t *__restrict__ hid)
{
    constexpr bool kSpread = (OPS & kOpSpread) != 0, kGather = (OPS & (kOpInterp | kOpGrad)) != 0;
    using Acc = typename AccType<T, MODE>::type;
    __shared__ uint32_t keys[kSpread ? kNodeSlots : 1];
    __shared__ Acc vals[kSpread ? 3 * kNodeSlots : 1];
    __shared__ T buf[kGather ? kNodePts : 1][27][NodeVals<OPS>::value];
    const NodeLane ln;
    const int64_t k = (int64_t)blockIdx.x * kNodePts + ln.slot;
    const bool have = ln.used && k < n;
    const int64_t kc = k < n ? k : n - 1;
    const T X[3] = {pos[3 * kc], pos[3 * kc + 1], pos[3 * kc + 2]};
    T F[3] = {T(0), T(0), T(0)};
    if (OPS & (kOpSpread | kOpGrad)) {
#pragma unroll
        for (int c = 0; c < 3; ++c) F[c] = force[3 * kc + c];
    }
    double scale = 0.0;
    if (kSpread && MODE == kModeFixed) {
        bool poison;
        scale = ldexp(1.0, fx_parts_shift<T>(fx, poison));
    }
    LdsSink<T, MODE, kNodeSlots> sink{keys, vals, fout, facc, scale};
    if (kSpread) {
        sink.clear();
        __syncthreads();
    }
    uint32_t I[3];
    bool ok = point_cell<T>(tv, X[0], X[1], X[2], I);
    uint32_t e = 0u;
    if (hid) ok = host_from_id(tv, hid[kc], e) && ok;
    else if (ok) e = descend(tv, I[0], I[1], I[2]);
    if (!ok) e = 0u;
    if ((OPS & kOpLocate) && have && ln.row == 0) ids[k] = ok ? (int32_t)(e & kIdMask) : -1;
    node_step<T, OPS, MODE, PER, kNodeSlots>(tv, ln, X, I, e, ok && have, have, F, k, field, vel, grad, sink, buf);
    if (kSpread) sink.flush();
}

// Ranges of sorted points (first sorted point, count), or every `pts` points
// of n when ranges is null: one spreading table per range.  word_host: the
// sort words hold the hosts (else block keys: the host is searched).
struct NodeRanges {
    const uint2 *ranges;
    const unsigned *count;
    int64_t n;
    int pts;
    bool word_host;
};

// Points of a range of a whole run: what the table holds the nodes of.  Points
// much rarer than leaves share few nodes (27 each), so one step's worth.  Sums
// added in FP64 (atomic_f64) are rounded at each add, in the table too: long
// ranges make long chains there, short ones more adds to device memory.  Steps
// that grow with the run keep them as exact as the tiles of an unsorted call or
// of a plan sorted by host (points in host order on 4,096 leaves, relative
// error of the field by tiles, 4 steps, these: 65 k 3.6e-16, 4.4e-16, 3.5e-16; 100 k
// 4.2e-16, 4.7e-16, 4.1e-16; spreading 50 k 49 -> 53 us, 100 k 67 -> 71).
constexpr int64_t kRangeStepPts = 50000;
inline int node_range_pts(const ot_tree *t, int64_t n, bool atomic_f64)
{
    if (4 * n < t->n_leaves) return kRangePts;
    return (atomic_f64 ? (int)std::max<int64_t>(1, std::min<int64_t>(4, n / kRangeStepPts)) : 4) * kRangePts;
}

template <typename T, int OPS, int MODE, bool PER>
__global__ __launch_bounds__(kRangeThreads) void k_node_ranges(TreeView tv, NodeRanges nr, unsigned *__restrict__ queue,
                                                               const uint64_t *__restrict__ kv,
                                                               const T *__restrict__ rec, const T *__restrict__ field,
                                                               T *__restrict__ vel, T *__restrict__ fout,
                                                               unsigned long long *__restrict__ facc, FxRef fx,
                                                               T *__restrict__ grad)
{
    constexpr bool kSpread = (OPS & kOpSpread) != 0, kGather = (OPS & (kOpInterp | kOpGrad)) != 0;
    constexpr int RS = (OPS & (kOpSpread | kOpGrad)) ? 6 : 3;
    using Acc = typename AccType<T, MODE>::type;
    __shared__ uint32_t keys[kSpread ? kRangeSlots : 1];
    __shared__ Acc vals[kSpread ? 3 * kRangeSlots : 1];
    __shared__ T buf[kGather ? kRangePts : 1][27][NodeVals<OPS>::value];
    __shared__ unsigned s_next;
    const NodeLane ln;
    const double scale = (kSpread && MODE == kModeFixed) ? fx_scale<T>(fx) : 0.0;
    LdsSink<T, MODE, kRangeSlots> sink{keys, vals, fout, facc, scale};
    if (kSpread) sink.clear();
    const unsigned nt = nr.ranges ? *nr.count : (unsigned)((nr.n + nr.pts - 1) / nr.pts);
    unsigned nxt = 0u;
    if (threadIdx.x == 0) nxt = atomicAdd(queue, 1u);
    for (;;) {
        if (threadIdx.x == 0) s_next = nxt;
        __syncthreads();
        const unsigned ti = s_next;
        if (ti >= nt) break;   // uniform
        int64_t start = (int64_t)ti * nr.pts, end = min(start + (int64_t)nr.pts, nr.n);
        if (nr.ranges) {
            start = nr.ranges[ti].x;
            end = start + nr.ranges[ti].y;
        }
        // the next step's word, position and force are loaded before this step's work
        auto load = [&](int64_t b, uint64_t &wd, T (&X)[3], T (&F)[3]) {
            const int64_t k = min(b + ln.slot, end - 1);
            wd = kv[k];
#pragma unroll
            for (int c = 0; c < 3; ++c) X[c] = rec[RS * k + c];
#pragma unroll
            for (int c = 0; c < 3; ++c) F[c] = RS == 6 ? rec[RS * k + 3 + c] : T(0);
        };
        uint64_t wn;
        T Xn[3], Fn[3];
        load(start, wn, Xn, Fn);
        for (int64_t b = start; b < end; b += kRangePts) {
            const uint64_t wd = wn;
            const T X[3] = {Xn[0], Xn[1], Xn[2]}, F[3] = {Fn[0], Fn[1], Fn[2]};
            load(b + kRangePts, wn, Xn, Fn);
            const bool have = ln.used && b + ln.slot < end;
            uint32_t I[3];
            const bool ok = point_cell<T>(tv, X[0], X[1], X[2], I);
            uint32_t e = 0u;
            if (ok) e = nr.word_host ? (uint32_t)(wd >> 32) : descend(tv, I[0], I[1], I[2]);
            node_step<T, OPS, MODE, PER, kRangeSlots>(tv, ln, X, I, e, ok && have, have, F, (int64_t)(uint32_t)wd, field,
                                                      vel, grad, sink, buf);
            if (kGather) __syncthreads();   // buf is free again
        }
        if (threadIdx.x == 0) nxt = atomicAdd(queue, 1u);
        if (kSpread) sink.flush();
        else __syncthreads();   // every thread has read s_next
    }
}

}  // namespace ot
