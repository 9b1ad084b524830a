// Multi-direct forcing of the immersed-boundary method (IBM subsection of
// Sec. 2.2): per iteration, interpolate the leaf velocity to the markers,
// form the marker force from the slip against the prescribed marker
// velocity, spread it back to the leaves and correct the leaf velocity.
//
// The markers do not move during the iterations, so once per call every
// marker's stencil is computed and kept: its 27 node leaves and weights, as
// the tracking kernel forms them (its own lookups and products, so the same
// values).  The leaves the stencils reach are listed, and the (marker, node)
// pairs grouped by listed leaf.  An iteration is then two passes without
// atomic adds: one over the markers (interpolation by gathering through the
// kept stencils, slip force, max |F|), one over the listed leaves (each sums
// its pairs' contributions, in FIXED mode as the rounded integers of plain
// spreading, and applies u += f / rho).  Every marker's and every leaf's
// arithmetic is that of the plain composition of the library's
// interpolation and spreading (FIXED: bit for bit; ATOMIC: each leaf's sum
// in FP64, rounded once).  Everything is enqueued on the caller's stream;
// the caller provides the workspace; no memset nodes, so the call can be
// captured in a graph.
#include <hip/hip_runtime.h>

#include <limits>
#include <type_traits>

#include "node_pass.h"
#include "ot_common.h"
#include "track_device.h"

namespace ot {
namespace {

constexpr int kNodes = 27;

// The items [0, m) of a grid-stride loop, shared out so that each of the 8 XCDs
// (workgroups go to them in turn) takes a contiguous eighth: neighbouring
// markers and leaves read each other's entries, which then stay in one L2.
struct Share {
    int64_t i, end, step;
    __device__ __forceinline__ Share(int64_t m, int per_block, int within)
    {
        const int parts = min((int)gridDim.x, 8), part = (int)blockIdx.x % parts;
        const int blocks = ((int)gridDim.x - part + parts - 1) / parts;   // of this part
        end = m * (part + 1) / parts;
        i = m * part / parts + (int64_t)((int)blockIdx.x / parts) * per_block + within;
        step = (int64_t)blocks * per_block;
    }
};

// max |F| of one iteration, and of the next: up to kMaxSlots slots each, every
// one in a cache line of its own, since atomics on one line serialise (16 slots
// in one line: 21 us a marker pass of 2,357 workgroups, 15 us of 1,024).
constexpr int kMaxSlots = 64, kMaxStride = 16;   // slots, words of 8 bytes
struct MaxSlots {
    unsigned long long *p;
    int slots;
    __device__ __forceinline__ unsigned long long *at(int it, int i) const
    {
        return p + (int64_t)kMaxStride * ((it & 1) * slots + i);
    }
};

// Everything the call adds to or marks, in one launch.
template <typename T>
__global__ __launch_bounds__(256) void k_mdf_clear(T *__restrict__ f_lag, int64_t m_pts, T *__restrict__ f_eul,
                                                   int64_t m_leaves, uint32_t *__restrict__ flags, int64_t n_flags,
                                                   uint32_t *__restrict__ cnt, int64_t n_cnt,
                                                   unsigned long long *__restrict__ maxb)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (f_lag)
        for (int64_t i = t; i < m_pts; i += step) f_lag[i] = T(0);
    if (f_eul)
        for (int64_t i = t; i < m_leaves; i += step) f_eul[i] = T(0);
    for (int64_t i = t; i < n_flags; i += step) flags[i] = 0u;
    for (int64_t i = t; i < n_cnt; i += step) cnt[i] = 0u;
    if (t < 2 * kMaxStride) maxb[t] = 0ull;
}

// Node leaves (-1: dropped at a wall, or no host) and weights of every marker,
// nine lanes a marker (its rows of three nodes): a marker's 27 lookups side by
// side and its entries stored next to each other.  66 k markers: 15 us; 24 with
// one thread a marker, which stored at a stride of 27 entries.
template <typename T, bool PER>
__global__ __launch_bounds__(kNodeThreads) void k_mdf_stencil(TreeView tv, int64_t n, const T *__restrict__ pos,
                                                              int32_t *__restrict__ leaf, T *__restrict__ wt,
                                                              uint32_t *__restrict__ flags)
{
    const NodeLane ln;
    const int64_t k = (int64_t)blockIdx.x * kNodePts + ln.slot;
    if (!ln.used || k >= n) return;
    const T X[3] = {pos[3 * k], pos[3 * k + 1], pos[3 * k + 2]};
    uint32_t I[3];
    const bool ok = point_cell<T>(tv, X[0], X[1], X[2], I);
    const uint32_t e = ok ? descend(tv, I[0], I[1], I[2]) : 0u;
    const int l = (int)((e >> kLevelShift) & 31u);
    NodeRow nr;
    node_row<PER>(tv, ln, I, l, ok, nr);
    T w[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T t, r;
        cell_offsets<T>(X[d] * (T)(1 << l), t, r);
        delta3<T>(t, r, w[d]);
    }
    const T wy = ln.oy == 0 ? w[1][0] : ln.oy == 1 ? w[1][1] : w[1][2];
    const T wz = ln.oz == 0 ? w[2][0] : ln.oz == 1 ? w[2][1] : w[2][2];
    const int64_t at = kNodes * k + 3 * ln.row;
#pragma unroll
    for (int ox = 0; ox < 3; ++ox) {
        const uint32_t id = nr.ent[ox] & kIdMask;
        leaf[at + ox] = nr.in[ox] ? (int32_t)id : -1;
        wt[at + ox] = w[0][ox] * wy * wz;
        if (nr.in[ox]) flags[id] = 1u;
    }
}

// hi (nullable): the scanned sums of the scan's 2,048-value blocks, added here.
__global__ __launch_bounds__(256) void k_compact(const uint32_t *__restrict__ flags, uint32_t *__restrict__ offs,
                                                 const uint32_t *__restrict__ hi, int64_t m, int32_t *__restrict__ list,
                                                 uint32_t *__restrict__ count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t o = offs[i] + (hi ? hi[i / kScanBlock] : 0u);
        if (flags[i]) {
            list[o] = (int32_t)i;
            offs[i] = o;   // read for flagged leaves only
        }
        if (i == m - 1) *count = o + flags[i];
    }
}

// Pairs per listed leaf (offs maps a flagged leaf to its list index).
__global__ __launch_bounds__(256) void k_pair_count(const int32_t *__restrict__ leaf, int64_t m,
                                                    const uint32_t *__restrict__ offs, uint32_t *__restrict__ cnt)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t l = leaf[i];
        if (l >= 0) atomicAdd(&cnt[offs[l]], 1u);
    }
}

// pairs[start[li] ..] = marker * kNodes + node of every pair reaching listed leaf
// li; left counts li's pairs down to none.
__global__ __launch_bounds__(256) void k_pair_fill(const int32_t *__restrict__ leaf, int64_t m,
                                                   const uint32_t *__restrict__ offs, const uint32_t *__restrict__ start,
                                                   uint32_t *__restrict__ left, uint32_t *__restrict__ pairs)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t l = leaf[i];
        if (l >= 0) {
            const uint32_t li = offs[l];
            pairs[start[li] + atomicSub(&left[li], 1u) - 1u] = (uint32_t)i;
        }
    }
}

// Per marker: U = sum over its kept nodes of w u[leaf] (the tracking
// kernel's order and operations), F = (target - U) / dt into fk, f_lag
// (nullable) += F, and max |F| (finite components) into iteration it's slots
// (none: not wanted).  Nine lanes a marker read its entries and gather; one lane per
// component then sums the 27 products from LDS in their order.  66 k markers: 10.6
// us, 15.5 with one thread a marker.
template <typename T>
__global__ __launch_bounds__(kNodeThreads) void k_mdf_markers(int64_t n, const int32_t *__restrict__ leaf,
                                                              const T *__restrict__ wt, const T *__restrict__ u,
                                                              const T *__restrict__ target, T *__restrict__ fk,
                                                              T *__restrict__ f_lag, T dt, MaxSlots mx, int it)
{
    __shared__ T buf[kNodePts][kNodes][4];   // weight (NaN: no node) and field row
    __shared__ unsigned long long wmax[kNodeThreads / 64];
    const NodeLane ln;
    unsigned long long best = 0;
    const Share sh(n, kNodePts, 0);
    for (int64_t b = sh.i; b < sh.end; b += sh.step) {   // uniform
        const int64_t k = b + ln.slot;
        const bool have = ln.used && k < sh.end;
        if (have) {
            const int64_t at = kNodes * k + 3 * ln.row;
            int32_t l[3];
            T w[3];
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                l[ox] = leaf[at + ox];
                w[ox] = wt[at + ox];
            }
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const int64_t j = 3 * (int64_t)(l[ox] < 0 ? 0 : l[ox]);
                T *c = buf[ln.slot][3 * ln.row + ox];
                c[0] = l[ox] < 0 ? std::numeric_limits<T>::quiet_NaN() : w[ox];
                c[1] = u[j];
                c[2] = u[j + 1];
                c[3] = u[j + 2];
            }
        }
        __syncthreads();
        if (have && ln.row < 3) {
            T U = T(0);
#pragma unroll
            for (int q = 0; q < kNodes; ++q) {
                const T w = buf[ln.slot][q][0];
                const T s = fma(w, buf[ln.slot][q][1 + ln.row], U);
                U = w == w ? s : U;
            }
            const int64_t i = 3 * k + ln.row;
            const T F = (target[i] - U) / dt;
            fk[i] = F;
            if (f_lag) f_lag[i] += F;
            if (isfinite(F)) best = std::max(best, abs_bits(F));
        }
        __syncthreads();   // buf is free again
    }
    if (!mx.slots) return;   // the same for every thread
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = std::max(best, (unsigned long long)__shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kNodeThreads / 64; ++w) best = std::max(best, wmax[w]);
        if (best) atomicMax(mx.at(it, (int)blockIdx.x % mx.slots), best);
    }
}

// Per listed leaf: the sum of its pairs' contributions, f_eul (nullable) += f
// and u += f / rho.  FIXED: rounded integers at the call's scale, so their
// order does not matter.  Four lanes share a leaf's pairs (a leaf's loads were
// one chain of dependent ones), each XCD a contiguous eighth of the leaves.  Bound
// by scattered reads of weights and forces: 66 k markers 16 us, 17.6 with one lane
// a leaf in any order.
template <typename T, bool FIXED>
__global__ __launch_bounds__(256) void k_mdf_leaves(const int32_t *__restrict__ list, const uint32_t *__restrict__ count,
                                                    const uint32_t *__restrict__ start, const uint32_t *__restrict__ pairs,
                                                    const T *__restrict__ wt, const T *__restrict__ fk, MaxSlots mx,
                                                    int it, int64_t n,
                                                    T *__restrict__ u, T *__restrict__ f_eul, T rho)
{
    const int64_t c = *count;
    double scale = 0.0, inv = 0.0;
    if constexpr (FIXED) {
        const int lane = (int)(threadIdx.x & 63);
        unsigned long long best = *mx.at(it, lane < mx.slots ? lane : 0);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) best = std::max(best, (unsigned long long)__shfl_xor(best, o, 64));
        const int s = fx_shift<T>(best, n);
        scale = ldexp(1.0, s);
        inv = ldexp(1.0, -s);
        if (blockIdx.x == 0 && (int)threadIdx.x < mx.slots) *mx.at(it + 1, (int)threadIdx.x) = 0ull;
    }
    using Acc = typename std::conditional<FIXED, unsigned long long, double>::type;
    const uint32_t sub = threadIdx.x & 3u;
    const Share sh(c, 64, (int)(threadIdx.x >> 2));
    // a leaf's four lanes leave the loop together
    for (int64_t i = sh.i; i < sh.end; i += sh.step) {
        Acc a[3] = {Acc(0), Acc(0), Acc(0)};
        const uint32_t end = start[i + 1];
#pragma unroll 2
        for (uint32_t p = start[i] + sub; p < end; p += 4u) {
            const uint32_t pr = pairs[p];
            const int64_t k = pr / kNodes;
            const T w = wt[pr];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if constexpr (FIXED) a[d] += fx_round_fma((double)w, (double)fk[3 * k + d] * scale);
                else a[d] += (double)w * (double)fk[3 * k + d];
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            a[d] += __shfl_xor(a[d], 1, 64);
            a[d] += __shfl_xor(a[d], 2, 64);
        }
        if (sub < 3u) {
            const Acc v = sub == 0u ? a[0] : sub == 1u ? a[1] : a[2];
            const int64_t j = 3 * (int64_t)list[i] + sub;
            const T fi = FIXED ? (T)((double)(long long)v * inv) : (T)v;
            u[j] += fi / rho;
            if (f_eul) f_eul[j] += fi;
        }
    }
}

unsigned grid_for(int64_t m) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((m + 255) / 256, 4096)); }

// Workspace layout (bytes, each part 256-aligned): kept node leaves and
// weights (27n each), marker forces (3n T), flags, offsets and list
// (n_leaves words each), count, scan scratch, pair counts and starts
// (min(n_leaves, 27n) + 1 words each), pairs (27n words), max |F| of two iterations.
struct MdfWork {
    int32_t *leaf, *list;
    void *wt, *fk;
    uint32_t *flags, *offs, *count, *tmp, *cnt, *start, *pairs;
    unsigned long long *maxb;
    int64_t lmax;
};

int64_t align256(int64_t b) { return (b + 255) & ~int64_t(255); }

int64_t mdf_layout(int64_t n, int64_t n_leaves, int64_t tsize, char *base, MdfWork *w)
{
    int64_t o = 0;
    auto take = [&](int64_t bytes) {
        char *p = base ? base + o : nullptr;
        o += align256(bytes);
        return p;
    };
    const int64_t lmax = std::min<int64_t>(n_leaves, kNodes * n);
    char *leaf = take(4 * kNodes * n), *wt = take(tsize * kNodes * n), *fk = take(3 * n * tsize);
    char *flags = take(4 * n_leaves), *offs = take(4 * n_leaves), *list = take(4 * n_leaves);
    char *count = take(4), *tmp = take(4 * scan_tmp_words(n_leaves + 1));
    char *cnt = take(4 * (lmax + 1)), *start = take(4 * (lmax + 1)), *pairs = take(4 * kNodes * n);
    char *maxb = take(8 * 2 * kMaxStride);
    if (w)
        *w = MdfWork{(int32_t *)leaf,      (int32_t *)list,  wt,
                     fk,                   (uint32_t *)flags, (uint32_t *)offs,
                     (uint32_t *)count,    (uint32_t *)tmp,   (uint32_t *)cnt,
                     (uint32_t *)start,    (uint32_t *)pairs, (unsigned long long *)maxb,
                     lmax};
    return o;
}

template <typename T>
int mdf(const ot_tree *t, T *field, const T *pos, const T *target, int64_t n, int n_iter, T dt, T rho, int mode,
        T *f_lag, T *f_eul, void *work, hipStream_t s)
{
    const int64_t m_pts = 3 * n, m_leaves = 3 * t->n_leaves, m_nodes = kNodes * n;
    MdfWork w;
    mdf_layout(n, t->n_leaves, sizeof(T), (char *)work, &w);
    T *wt = (T *)w.wt, *fk = (T *)w.fk;
    if (n_iter == 0 || n == 0) {
        if (f_lag) hipLaunchKernelGGL(k_fill<T>, dim3(grid_for(m_pts)), dim3(256), 0, s, f_lag, m_pts, T(0));
        if (f_eul) hipLaunchKernelGGL(k_fill<T>, dim3(grid_for(m_leaves)), dim3(256), 0, s, f_eul, m_leaves, T(0));
        OT_HIP(hipGetLastError());
        return OT_OK;
    }
    // stencils kept, leaves listed, pairs grouped by listed leaf: once
    hipLaunchKernelGGL(k_mdf_clear<T>, dim3(grid_for(std::max(m_leaves, m_pts) / 4)), dim3(256), 0, s, f_lag, m_pts,
                       f_eul, m_leaves, w.flags, t->n_leaves, w.cnt, w.lmax + 1, w.maxb);
    const dim3 gm((unsigned)((n + kNodePts - 1) / kNodePts));
    if (t->view.periodic)
        hipLaunchKernelGGL((k_mdf_stencil<T, true>), gm, dim3(kNodeThreads), 0, s, t->view, n, pos, w.leaf, wt, w.flags);
    else
        hipLaunchKernelGGL((k_mdf_stencil<T, false>), gm, dim3(kNodeThreads), 0, s, t->view, n, pos, w.leaf, wt, w.flags);
    const uint32_t *hi = exclusive_scan_split(w.flags, w.offs, t->n_leaves, w.tmp, s);
    hipLaunchKernelGGL(k_compact, dim3(grid_for(t->n_leaves)), dim3(256), 0, s, w.flags, w.offs, hi, t->n_leaves,
                       w.list, w.count);
    hipLaunchKernelGGL(k_pair_count, dim3(grid_for(m_nodes)), dim3(256), 0, s, w.leaf, m_nodes, w.offs, w.cnt);
    exclusive_scan(w.cnt, w.start, w.lmax + 1, w.tmp, s);
    hipLaunchKernelGGL(k_pair_fill, dim3(grid_for(m_nodes)), dim3(256), 0, s, w.leaf, m_nodes, w.offs, w.start,
                       w.cnt, w.pairs);
    OT_HIP(hipGetLastError());
    const bool fixed = mode == OT_SPREAD_FIXED;
    const unsigned gl = grid_for(4 * w.lmax);
    // (66 k markers: 11.6 us at 4 workgroups per CU, 10.6 at 8, 11.6 at 16)
    const unsigned gk = (unsigned)std::min<int64_t>((n + kNodePts - 1) / kNodePts, 8 * t->cus);
    // the maxima's slots: the pair counts, all counted down to 0 by now, or in
    // small calls one slot
    MaxSlots mx{(unsigned long long *)w.cnt,
                (int)std::min<int64_t>(kMaxSlots, (w.lmax + 1) / (4 * kMaxStride))};
    if (mx.slots < 1) mx = MaxSlots{w.maxb, 1};
    if (!fixed) mx.slots = 0;
    for (int it = 0; it < n_iter; ++it) {
        hipLaunchKernelGGL(k_mdf_markers<T>, dim3(gk), dim3(kNodeThreads), 0, s, n, (const int32_t *)w.leaf,
                           (const T *)wt, (const T *)field, target, fk, f_lag, dt, mx, it);
        const auto leaves = fixed ? k_mdf_leaves<T, true> : k_mdf_leaves<T, false>;
        hipLaunchKernelGGL(leaves, dim3(gl), dim3(256), 0, s, (const int32_t *)w.list, (const uint32_t *)w.count,
                           (const uint32_t *)w.start, (const uint32_t *)w.pairs, (const T *)wt, (const T *)fk, mx, it,
                           n, field, f_eul, rho);
        OT_HIP(hipGetLastError());
    }
    return OT_OK;
}

}  // namespace
}  // namespace ot

using namespace ot;

extern "C" int64_t ot_mdf_workspace_bytes(const ot_tree *tree, int64_t n, int32_t dtype)
{
    if (!tree || n < 0 || (dtype != OT_F32 && dtype != OT_F64)) return -1;
    return mdf_layout(n, tree->n_leaves, dtype == OT_F32 ? 4 : 8, nullptr, nullptr);
}

extern "C" int ot_mdf(const ot_tree *tree, void *field, const void *pos, const void *target, int32_t dtype, int64_t n,
                      int32_t n_iter, double dt, double rho, int32_t mode, void *force_lag, void *force_eul,
                      void *work, void *stream)
{
    if (!tree) return fail(OT_ERR_INVALID, "ot_mdf: tree is NULL");
    if (dtype != OT_F32 && dtype != OT_F64) return fail(OT_ERR_INVALID, "dtype must be OT_F32 or OT_F64");
    if (n < 0 || n_iter < 0) return fail(OT_ERR_INVALID, "ot_mdf: n and n_iter must be >= 0");
    if (mode != OT_SPREAD_ATOMIC && mode != OT_SPREAD_FIXED) return fail(OT_ERR_INVALID, "bad spread mode");
    if (!(dt > 0.0) || !(rho > 0.0)) return fail(OT_ERR_INVALID, "ot_mdf: dt and rho must be positive");
    if (!field || !work || (n > 0 && (!pos || !target)))
        return fail(OT_ERR_INVALID, "ot_mdf: field, work, pos or target is NULL");
    if ((uintptr_t)work & 7) return fail(OT_ERR_INVALID, "ot_mdf: work must be 8-byte aligned");
    if (n > (int64_t)(UINT32_MAX / kNodes)) return fail(OT_ERR_CAPACITY, "ot_mdf: at most 159,072,862 markers");
    hipStream_t s = (hipStream_t)stream;
    if (dtype == OT_F32)
        return mdf<float>(tree, (float *)field, (const float *)pos, (const float *)target, n, n_iter, (float)dt,
                          (float)rho, mode, (float *)force_lag, (float *)force_eul, work, s);
    return mdf<double>(tree, (double *)field, (const double *)pos, (const double *)target, n, n_iter, dt, rho, mode,
                       (double *)force_lag, (double *)force_eul, work, s);
}
