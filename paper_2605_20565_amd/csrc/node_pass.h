// Node-parallel pass for small point sets: nine lanes per point, each with one
// x-row of three stencil nodes.
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

#include "ot_common.h"
#include "track_device.h"

namespace ot {

constexpr int kNodeLanes = 9;                                        // lanes per point: (oy, oz)
constexpr int kNodeThreads = 256;
constexpr int kNodeWavePts = 64 / kNodeLanes;                        // 7; lane 63 idles
constexpr int kNodePts = kNodeWavePts * (kNodeThreads / 64);         // 28 points per workgroup
constexpr int kNodeSlots = 1024;                                     // spreading table (28 x 27 nodes at most)

template <typename T, int OPS, int MODE, bool PER>
__global__ __launch_bounds__(kNodeThreads) void k_nodes(TreeView tv, int64_t n, const T *__restrict__ pos,
                                                        const T *__restrict__ field, const T *__restrict__ force,
                                                        int32_t *__restrict__ ids, T *__restrict__ vel,
                                                        T *__restrict__ fout, unsigned long long *__restrict__ facc,
                                                        const FxState *__restrict__ fx, T *__restrict__ grad,
                                                        const int32_t *__restrict__ hid)
{
    constexpr bool kInterp = (OPS & kOpInterp) != 0, kGrad = (OPS & kOpGrad) != 0, kSpread = (OPS & kOpSpread) != 0;
    constexpr bool kGather = kInterp || kGrad;
    constexpr int kVals = kGrad ? 6 : 4;   // per node: weight and field row; gradient: two factors per axis
    using Acc = typename AccType<T, MODE>::type;
    __shared__ uint32_t keys[kSpread ? kNodeSlots : 1];
    __shared__ Acc vals[kSpread ? 3 * kNodeSlots : 1];
    __shared__ T buf[kGather ? kNodePts : 1][27][kVals];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int p = lane / kNodeLanes, row = lane - kNodeLanes * p;
    const int oy = row % 3, oz = row / 3;
    const int slot = wid * kNodeWavePts + (p < kNodeWavePts ? p : 0);
    const int64_t k = (int64_t)blockIdx.x * kNodePts + slot;
    const bool have = p < kNodeWavePts && k < n;
    const int64_t kc = k < n ? k : n - 1;
    const T X[3] = {pos[3 * kc], pos[3 * kc + 1], pos[3 * kc + 2]};
    T F[3] = {T(0), T(0), T(0)};
    if (kSpread || kGrad) {
#pragma unroll
        for (int c = 0; c < 3; ++c) F[c] = force[3 * kc + c];
    }
    double scale = 0.0;
    if (kSpread && MODE == kModeFixed) {
        double inv;
        bool poison;
        fx_scale<T>(fx, n, scale, inv, poison);
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
    if ((OPS & kOpLocate) && have && row == 0) ids[k] = ok ? (int32_t)(e & kIdMask) : -1;
    ok = ok && have;

    // the stencil's 1-D weights, and this lane's three nodes
    const int l = (int)((e >> kLevelShift) & 31u), sh = tv.L - l, rsh = tv.L - tv.lev[0];
    const int32_t M = 1 << l;
    const uint32_t half = sh > 0 ? 1u << (sh - 1) : 0u;
    const T sc = (T)M;
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
    uint32_t ent[3], root[3], N[3][3];
    bool in[3];
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) {
        const int o[3] = {ox, oy, oz};
        in[ox] = ok;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int32_t c = (int32_t)(I[d] >> sh) + o[d] - 1;
            if (PER) c &= M - 1;
            else in[ox] = in[ox] && c >= 0 && c < M;
            N[ox][d] = ((uint32_t)c << sh) | half;
        }
        if (!in[ox]) N[ox][0] = N[ox][1] = N[ox][2] = 0u;
        root[ox] = interleave3(N[ox][0] >> rsh, N[ox][1] >> rsh, N[ox][2] >> rsh);
        ent[ox] = ld_table(tv, root[ox]);
    }
    uint32_t sub[3];
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) sub[ox] = ld_table(tv, step1_index(tv, ent[ox], N[ox][0], N[ox][1], N[ox][2]));
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) {
        if (ent[ox] & kSplit) ent[ox] = sub[ox];
        if (ent[ox] & kSplit) ent[ox] = descend_from_level2(tv, ent[ox], N[ox][0], N[ox][1], N[ox][2]);
    }
    // a lane's own row of weights, picked without indexing registers by lane
    const T wy = oy == 0 ? w[1][0] : oy == 1 ? w[1][1] : w[1][2];
    const T wz = oz == 0 ? w[2][0] : oz == 1 ? w[2][1] : w[2][2];

    if (kGather) {
        T f[3][3];
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
            const int64_t j = 3 * (int64_t)(in[ox] ? ent[ox] & kIdMask : 0u);
#pragma unroll
            for (int c = 0; c < 3; ++c) f[ox][c] = field[j + c];
        }
        if (kInterp) {
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                T *b = buf[slot][3 * row + ox];
                if (p < kNodeWavePts) {
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
                vel[3 * k + row] = ok ? U : T(0);
            }
            if (kGrad) __syncthreads();
        }
        if constexpr (kGrad) {
            const T dy = oy == 0 ? dw[1][0] : oy == 1 ? dw[1][1] : dw[1][2];
            const T dz = oz == 0 ? dw[2][0] : oz == 1 ? dw[2][1] : dw[2][2];
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const T dot = fma(F[0], f[ox][0], fma(F[1], f[ox][1], F[2] * f[ox][2]));
                T *b = buf[slot][3 * row + ox];
                if (p < kNodeWavePts) {
                    b[0] = in[ox] ? dot * dw[0][ox] : T(0);
                    b[1] = wy * wz;
                    b[2] = in[ox] ? dot * w[0][ox] : T(0);
                    b[3] = dy * wz;
                    b[4] = b[2];
                    b[5] = wy * dz;
                }
            }
            __syncthreads();
            if (row < 3 && have) {
                T G = T(0);
#pragma unroll
                for (int q = 0; q < 27; ++q) G = fma(buf[slot][q][2 * row], buf[slot][q][2 * row + 1], G);
                grad[3 * k + row] = ok ? G : T(0);
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
                const uint32_t old = atomicCAS(&keys[at[ox]], 0u, leaf + 1u);
                hit[ox] = old == 0u || old == leaf + 1u;
            }
        }
#pragma unroll
        for (int ox = 0; ox < 3; ++ox) {
            if (!in[ox]) continue;
            const T ww = w[0][ox] * wy * wz;
            Acc a[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c] = to_acc<T, MODE>(ww, F[c], scale);
            if (hit[ox]) {
#pragma unroll
                for (int c = 0; c < 3; ++c) atomicAdd(&vals[3 * at[ox] + c], a[c]);
            } else {
                sink.add_probing(ent[ox] & kIdMask, at[ox], a[0], a[1], a[2]);
            }
        }
        sink.flush();
    }
}

}  // namespace ot
