// Host-cell search, interpolation, spreading and the position gradient.
//
// One thread per Lagrangian point.  A point's integer cell is floor(x 2^L)
// in FP64 (so that a face decision never flips between precisions), its host
// leaf comes from the descent table (Sec. 3.2 / Algorithm 1 semantics), and
// the 3x3x3 stencil at the host level uses the 3-point delta function of
// Sec. 2.2.  Interpolation gathers the 27 node values; spreading scatters
// w F to the same 27 node leaves (atomics in the working precision, or
// int64 fixed point for order-independent sums).
#include <hip/hip_runtime.h>

#include "batch_plan.h"
#include "memory.h"
#include "node_pass.h"
#include "ot_common.h"
#include "track_device.h"

namespace ot {

// Launch of the plain kernels for one (precision, mode); instantiated in
// track_inst.hip (track_kernels.h).
template <typename T, int MODE>
int dispatch_ops(int ops, const ot_tree *t, dim3 g, dim3 b, int64_t tile, hipStream_t s, int64_t n, const void *pos,
                 const void *field, const void *force, int32_t *ids, void *vel, void *fout, void *grad,
                 const FxWs &ws, const int32_t *hid);

// Launch of the node-parallel pass; instantiated in node_inst.hip (node_pass.h).
template <typename T, int MODE>
int dispatch_nodes(int ops, const ot_tree *t, hipStream_t s, int64_t n, const void *pos, const void *field,
                   const void *force, int32_t *ids, void *vel, void *fout, void *grad, const FxWs &ws,
                   const int32_t *hid);

// A plain call as one run of a sorted plan (batch.hip).
int sorted_pass(const ot_tree *t, int ops, const void *field, const void *force, const void *pos, int dtype, int64_t n,
                int mode, int accumulate, int32_t *ids, void *vel, void *fout, void *grad, void *work, hipStream_t s,
                bool &handled);

constexpr int kMaxPointsPerThread = 4;

// Unsorted point sets up to these sizes take the node-parallel pass
// (node_pass.h).  Measured, FP32, random points on 38 k leaves, kernel alone,
// per-point pass against this one.  Interpolation: 1 k points 6.6 -> 4.5 us, 10 k
// 7.1 -> 4.9, 25 k 8.4 -> 5.0, 49 k 9.8 -> 7.4 (with the gradient 10.1 -> 11.1, and
// slower on larger trees from 25 k).  Spreading: 1 k 37 -> 9.2 us, 10 k 49 -> 18,
// 49 k 174 -> 61; calls that may not sort take it up to 65,535 points (from
// there the per-point pass takes tiles of 128 points with the large table, and
// markers in order on few leaves are faster there: 100 k 66 against 134 us a
// call).  A whole fused FP32 fixed-point call on 11 k points: 53.5 -> 25.9 us
// (three launches instead of five).
constexpr int64_t kNodesMaxSpread = 65535;   // sums in FP32 apart (nodes_max)
constexpr int64_t kNodesMaxGather = 16384;
// Trees of so few leaves that the smallest spreading table holds them all: the
// per-point pass then adds a leaf's sum to device memory once a workgroup in
// any order of the points, and sorting gains nothing (512 leaves, random
// points, fixed point, per-point pass against sorted: 100 k 47 against 59 us,
// 1 M 100 against 203, 4 M 294 against 696).  The node-parallel pass saves two
// launches of fixed-point calls (2 k points 21 -> 17 us, 16 k 23 against 29) and
// none of atomic ones, whose FP64 sums it makes less exact (8 k points 4.5e-16 ->
// 5.6e-16, 50 k 9.5e-16 -> 1.28e-15).
static_assert(kFewLeaves == kSmallSlots, "every leaf has a slot of its own");
constexpr int64_t kNodesMaxFewLeaves = 8192;
// Larger sets are sorted first, as a sorted plan does, when the call spreads,
// searches the hosts itself and may allocate.  What that gains depends on the
// order of the points, which nothing tells before the call: random ones fill
// an unsorted workgroup's spreading table many times over, those in order do
// not.  Unsorted against sorted, us a call on 38 k leaves, spreading in fixed
// point FP32: random points 65 k 95 (node pass) and 58, 100 k 238 and 64, 200 k
// 600 and 91, 1 M 3400 and 168; markers in order 65 k 86 and 56, 100 k 65 and 64,
// 200 k 86 and 93, 400 k 128 and 129, 1 M 243 and 187; points in host order 65 k
// 26 and 58, 100 k 46 and 63, 200 k 72 and 91, 400 k 174 and 127.  The lines lie
// where random points gain by half (kSortMinSpread); points in order lose up to
// some 400 k, and programs that keep them so have their hosts' ids to give,
// which keeps a call unsorted.  FP64 with gathers, whose ranges are slower,
// sort where the node pass ends (forward and backward of random points 65 k 102
// and 85, 100 k 247 and 95; markers in order 100 k 70 and 96, host order 48 and
// 95); sums in FP32, which do not take the node pass, from kSortMinF32Sums
// (random points 40 k 157 and 54, markers in order 88 and 48, host order 40 and
// 54).  Calls that only gather take their points as they are: sorting
// would gain with random points on large trees what it would lose with points
// in host order, as particles are kept (interpolation of 10^7 points, FP32, on
// 2.7 M leaves 2743 -> 702 us and 302 -> 535, on 38 k leaves 1175 -> 657 and 179 ->
// 522), and nothing tells the two apart before the call.  Programs with points
// in random order have sorted plans.

// Prepare the spreading target before a pass: zero the output (atomic mode,
// overwrite) or the fixed-point accumulators and compute the scale.
namespace {

// Zero n 64-bit words at a and, in block 0, m 32-bit words at b: one launch
// for the fixed-point workspace (its header first, then the accumulators)
// and a batch plan's counters.
__global__ void k_zero2(unsigned long long *__restrict__ a, int64_t n, unsigned *__restrict__ b, int64_t m)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0ull;
    if (b && blockIdx.x == 0)
        for (int64_t i = threadIdx.x; i < m; i += blockDim.x) b[i] = 0u;
}

// Small calls: zero n 64-bit words at a, and the max |F| of this workgroup's
// share of the m force components into parts (workgroups 0 .. kFxParts - 1).
template <typename T>
__global__ __launch_bounds__(256) void k_zero_max(unsigned long long *__restrict__ a, int64_t n,
                                                  const T *__restrict__ f, int64_t m,
                                                  unsigned long long *__restrict__ parts)
{
    if ((int)blockIdx.x >= kFxParts) {
        const int64_t step = (int64_t)(gridDim.x - kFxParts) * blockDim.x;
        for (int64_t i = (blockIdx.x - kFxParts) * (int64_t)blockDim.x + threadIdx.x; i < n; i += step) a[i] = 0ull;
        return;
    }
    __shared__ unsigned long long wmax[4];
    unsigned long long best = 0ull;
    constexpr int kU = 8;   // loads in flight per thread, at clamped indices
    const int64_t step = (int64_t)kFxParts * 256;
    for (int64_t i0 = blockIdx.x * (int64_t)256 + threadIdx.x; i0 < m; i0 += kU * step) {
        T v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = f[i0 + u * step < m ? i0 + u * step : i0];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const unsigned long long b = isfinite(v[u]) ? abs_bits(v[u]) : 0ull;
            best = std::max(best & 0x7FFFFFFFFFFFFFFFull, b) | (best & 0x8000000000000000ull) |
                   (isfinite(v[u]) ? 0ull : 0x8000000000000000ull);
        }
    }
    auto join = [](unsigned long long x, unsigned long long y) {
        return std::max(x & 0x7FFFFFFFFFFFFFFFull, y & 0x7FFFFFFFFFFFFFFFull) | ((x | y) & 0x8000000000000000ull);
    };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = join(best, (unsigned long long)__shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = join(join(wmax[0], wmax[1]), join(wmax[2], wmax[3]));
}

template <typename T>
void nodes_begin(const ot_tree *t, const FxWs &ws, const void *force, int64_t n, hipStream_t s)
{
    const int64_t n3 = t->n_leaves * 3;
    const unsigned gz = (unsigned)std::min<int64_t>((n3 + 255) / 256, 1024);
    hipLaunchKernelGGL(k_zero_max<T>, dim3(kFxParts + gz), dim3(256), 0, s, ws.acc, n3, (const T *)force, 3 * n,
                       ws.fx->parts);
}

template <typename T>
void nodes_end(const ot_tree *t, const FxWs &ws, int accumulate, void *fout, int64_t n, hipStream_t s)
{
    const int64_t n3 = t->n_leaves * 3;
    const unsigned gb = (unsigned)std::min<int64_t>((n3 + 255) / 256, 8192);
    hipLaunchKernelGGL((k_fx_finalize<T, true>), dim3(gb), dim3(256), 0, s, ws.acc, (T *)fout, n3, FxRef{ws.fx, n},
                       accumulate);
}

}  // namespace

int spread_begin(const ot_tree *t, const FxWs &ws, int dtype, int mode, int accumulate, void *fout, hipStream_t s,
                 unsigned *counters, int64_t n_counters)
{
    const int64_t n3 = t->n_leaves * 3;
    if (mode == OT_SPREAD_ATOMIC) {
        if (!accumulate) {
            if (dtype == OT_F32) hipLaunchKernelGGL(k_fill<float>, dim3(1024), dim3(256), 0, s, (float *)fout, n3, 0.0f);
            else hipLaunchKernelGGL(k_fill<double>, dim3(1024), dim3(256), 0, s, (double *)fout, n3, 0.0);
        }
        if (counters) hipLaunchKernelGGL(k_fill<unsigned>, dim3(1), dim3(64), 0, s, counters, n_counters, 0u);
    } else {
        // the whole header (max |F|, the non-finite flag) and the accumulators
        // after it, and the counters
        hipLaunchKernelGGL(k_zero2, dim3(1024), dim3(256), 0, s, (unsigned long long *)ws.fx,
                           kFxHeader / 8 + n3, counters, n_counters);
    }
    OT_HIP(hipGetLastError());
    return OT_OK;
}

int spread_max(const FxWs &ws, int dtype, int mode, const void *force, int64_t n, hipStream_t s)
{
    const int64_t m = n * 3;
    if (mode != OT_SPREAD_FIXED || !force || m <= 0) return OT_OK;
    unsigned gb = (unsigned)std::min<int64_t>((m + 1023) / 1024, 1024);
    if (dtype == OT_F32)
        hipLaunchKernelGGL(k_maxabs<float>, dim3(gb), dim3(256), 0, s, (const float *)force, m, &ws.fx->maxbits);
    else
        hipLaunchKernelGGL(k_maxabs<double>, dim3(gb), dim3(256), 0, s, (const double *)force, m, &ws.fx->maxbits);
    OT_HIP(hipGetLastError());
    return OT_OK;
}

int spread_epilogue(const ot_tree *t, const FxWs &ws, int dtype, int mode, int accumulate, void *fout, int64_t n,
                    hipStream_t s)
{
    if (mode != OT_SPREAD_FIXED) return OT_OK;
    const int64_t n3 = t->n_leaves * 3;
    const unsigned gb = (unsigned)std::min<int64_t>((n3 + 255) / 256, 8192);
    const FxRef fx{ws.fx, n};
    if (dtype == OT_F32)
        hipLaunchKernelGGL((k_fx_finalize<float, false>), dim3(gb), dim3(256), 0, s, ws.acc, (float *)fout, n3, fx,
                           accumulate);
    else
        hipLaunchKernelGGL((k_fx_finalize<double, false>), dim3(gb), dim3(256), 0, s, ws.acc, (double *)fout, n3, fx,
                           accumulate);
    OT_HIP(hipGetLastError());
    return OT_OK;
}

namespace {
__global__ void k_wide_finalize(const double *__restrict__ acc, float *__restrict__ out, int64_t n3, int accumulate)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n3; i += (int64_t)gridDim.x * blockDim.x) {
        const double v = acc[i];
        if (!accumulate) out[i] = (float)v;
        else if (v != 0.0) out[i] = (float)((double)out[i] + v);
    }
}
}  // namespace

int wide_epilogue(const ot_tree *t, const double *acc, int accumulate, float *fout, hipStream_t s)
{
    const int64_t n3 = t->n_leaves * 3;
    hipLaunchKernelGGL(k_wide_finalize, dim3((unsigned)std::min<int64_t>((n3 + 255) / 256, 8192)), dim3(256), 0, s, acc,
                       fout, n3, accumulate);
    OT_HIP(hipGetLastError());
    return OT_OK;
}

FxWs fx_ws(void *work)
{
    FxWs w;
    w.fx = (FxState *)work;
    w.acc = work ? (unsigned long long *)((char *)work + kFxHeader) : nullptr;
    return w;
}

int check_common(const ot_tree *t, int dtype, int64_t n, const void *pos)
{
    if (!t) return fail(OT_ERR_INVALID, "tree is NULL");
    if (dtype != OT_F32 && dtype != OT_F64) return fail(OT_ERR_INVALID, "dtype must be OT_F32 or OT_F64");
    if (n < 0) return fail(OT_ERR_INVALID, "n < 0");
    if (n > 0 && !pos) return fail(OT_ERR_INVALID, "pos is NULL");
    if (n > (int64_t(1) << 40)) return fail(OT_ERR_CAPACITY, "too many points");
    return OT_OK;
}

namespace {

// A small call's pass: three launches with fixed-point spreading.
template <typename T>
int nodes_pass(const ot_tree *t, int ops, const void *field, const void *force, const void *pos, int dtype, int64_t n,
               int mode, int accumulate, int32_t *ids, void *vel, void *fout, void *grad, const FxWs &ws,
               const int32_t *hid, hipStream_t s)
{
    const bool spread = (ops & kOpSpread) != 0, fixed = spread && mode == OT_SPREAD_FIXED;
    int rc = OT_OK;
    if (fixed) nodes_begin<T>(t, ws, force, n, s);
    else if (spread) rc = spread_begin(t, ws, dtype, mode, accumulate, fout, s);
    if (!rc)
        rc = fixed ? dispatch_nodes<T, kModeFixed>(ops, t, s, n, pos, field, force, ids, vel, fout, grad, ws, hid)
                   : dispatch_nodes<T, kModeAtomic>(ops, t, s, n, pos, field, force, ids, vel, fout, grad, ws, hid);
    if (!rc && fixed) nodes_end<T>(t, ws, accumulate, fout, n, s);
    OT_HIP(hipGetLastError());
    return rc;
}

// Enough workgroups to give every CU two, when there are points for them:
// small sets get narrower workgroups and one point per thread (their time is
// latency, not throughput); large ones up to kMaxPointsPerThread points per
// thread.
void track_shape(const ot_tree *t, int64_t n, int &threads, int64_t &tile)
{
    const int64_t want = 2 * (int64_t)t->cus;
    threads = 256;
    while (threads > 64 && (n + threads - 1) / threads < want) threads >>= 1;
    tile = threads * std::max<int64_t>(1, std::min<int64_t>(kMaxPointsPerThread, n / ((int64_t)threads * want)));
}

// Most points for which an unsorted call takes the node-parallel pass.  Sums in
// FP32 take the pass with the fewest adds to a leaf: workgroups of 28 points
// had made them up to 1.3 times less exact (16 k markers in order: 1.6e-7 ->
// 2.1e-7).
int64_t nodes_max(const ot_tree *t, int ops, int dtype, int mode)
{
    if (!(ops & ~kOpLocate)) return 0;
    if (!(ops & kOpSpread)) return kNodesMaxGather;
    if (t->n_leaves <= kFewLeaves) return mode == OT_SPREAD_FIXED ? kNodesMaxFewLeaves : 0;
    return mode == OT_SPREAD_ATOMIC && dtype == OT_F32 ? 0 : kNodesMaxSpread;
}

// The pass's kernel alone, no clearing, scale or conversion around it.
int launch_ops(const ot_tree *t, int ops, const void *field, const void *force, const void *pos, int dtype, int64_t n,
               int mode, int32_t *ids, void *vel, void *fout, void *grad, const FxWs &ws, const int32_t *hid,
               hipStream_t s)
{
    int rc = OT_OK;
    if (n > 0) {
        int threads;
        int64_t tile;
        track_shape(t, n, threads, tile);
        dim3 b(threads), g((unsigned)((n + tile - 1) / tile));
        if (dtype == OT_F32)
            rc = mode == OT_SPREAD_FIXED
                     ? dispatch_ops<float, kModeFixed>(ops, t, g, b, tile, s, n, pos, field, force, ids, vel, fout, grad,
                                                       ws, hid)
                     : dispatch_ops<float, kModeAtomic>(ops, t, g, b, tile, s, n, pos, field, force, ids, vel, fout,
                                                        grad, ws, hid);
        else
            rc = mode == OT_SPREAD_FIXED
                     ? dispatch_ops<double, kModeFixed>(ops, t, g, b, tile, s, n, pos, field, force, ids, vel, fout,
                                                        grad, ws, hid)
                     : dispatch_ops<double, kModeAtomic>(ops, t, g, b, tile, s, n, pos, field, force, ids, vel, fout,
                                                         grad, ws, hid);
        if (rc) return rc;
        OT_HIP(hipGetLastError());
    }
    return OT_OK;
}

// One pass over the points with the ops in `ops` (OT_OP_* bits, or the
// gradient with at most one of interpolation and spreading).  hid: the
// caller's host ids (nullable).  work: the fixed-point spreading workspace
// (FIXED spreading only; NULL: allocated on the stream for this call).
int run_pass(const ot_tree *t, int ops, const void *field, const void *force, const void *pos, int dtype, int64_t n,
             int mode, int accumulate, int32_t *ids, void *vel, void *fout, void *grad, const int32_t *hid,
             void *work, hipStream_t s, bool may_sort = true)
{
    int rc = check_common(t, dtype, n, pos);
    if (rc) return rc;
    const bool ops_ok = (ops > 0 && ops <= 7) || ops == kOpGrad || ops == (kOpGrad | kOpInterp) ||
                        ops == (kOpGrad | kOpSpread);
    if (!ops_ok) return fail(OT_ERR_INVALID, "ops must be a non-empty combination of OT_OP_* bits");
    if ((ops & kOpLocate) && n > 0 && !ids) return fail(OT_ERR_INVALID, "ids is NULL");
    if ((ops & kOpInterp) && ((n > 0 && !vel) || !field)) return fail(OT_ERR_INVALID, "field or vel is NULL");
    if ((ops & kOpGrad) && ((n > 0 && (!grad || !force)) || !field))
        return fail(OT_ERR_INVALID, "field, vector or gradient output is NULL");
    const bool spread = (ops & kOpSpread) != 0;
    if (spread) {
        if ((n > 0 && !force) || !fout) return fail(OT_ERR_INVALID, "force or field_out is NULL");
        if (mode != OT_SPREAD_ATOMIC && mode != OT_SPREAD_FIXED) return fail(OT_ERR_INVALID, "bad spread mode");
    }
    if (work && ((uintptr_t)work & 255u)) return fail(OT_ERR_INVALID, "work must be 256-byte aligned");
    void *owned = nullptr;
    if (spread && mode == OT_SPREAD_FIXED && !work) {
        hipError_t e = device_malloc_async(t->device, &owned, (size_t)spread_ws_bytes(t->n_leaves), s);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(OT_ERR_OOM, "fixed-point spreading workspace");
        }
        work = owned;
    }
    const FxWs ws = fx_ws(spread && mode == OT_SPREAD_FIXED ? work : nullptr);
    if (may_sort && !hid && plain_sorts(t, n, ops, dtype, mode)) {
        bool handled;
        rc = sorted_pass(t, ops, field, force, pos, dtype, n, mode, accumulate, ids, vel, fout, grad, work, s, handled);
        if (handled) {
            if (owned) (void)hipFreeAsync(owned, s);
            return rc;
        }
    }
    if (n > 0 && n <= nodes_max(t, ops, dtype, mode)) {
        rc = dtype == OT_F32 ? nodes_pass<float>(t, ops, field, force, pos, dtype, n, mode, accumulate, ids, vel, fout,
                                                 grad, ws, hid, s)
                             : nodes_pass<double>(t, ops, field, force, pos, dtype, n, mode, accumulate, ids, vel, fout,
                                                  grad, ws, hid, s);
        if (owned) (void)hipFreeAsync(owned, s);
        return rc;
    }
    if (spread) rc = spread_begin(t, ws, dtype, mode, accumulate, fout, s);
    if (!rc && spread) rc = spread_max(ws, dtype, mode, force, n, s);
    if (!rc) rc = launch_ops(t, ops, field, force, pos, dtype, n, mode, ids, vel, fout, grad, ws, hid, s);
    if (!rc && spread) rc = spread_epilogue(t, ws, dtype, mode, accumulate, fout, n, s);
    if (owned) (void)hipFreeAsync(owned, s);
    return rc;
}

}  // namespace

// A plain call as it is, unsorted (a plan of few points).
int plain_pass(const ot_tree *t, int ops, const void *field, const void *force, const void *pos, int dtype, int64_t n,
               int mode, int32_t *ids, void *vel, void *fout, void *grad, void *work, hipStream_t s)
{
    return run_pass(t, ops, field, force, pos, dtype, n, mode, 0, ids, vel, fout, grad, nullptr, work, s, false);
}

// Workgroups of plain_pass, one a tile.
int64_t plain_tiles(const ot_tree *t, int ops, int dtype, int64_t n, int mode)
{
    if (n <= nodes_max(t, ops, dtype, mode)) return (n + kNodePts - 1) / kNodePts;
    int threads;
    int64_t tile;
    track_shape(t, n, threads, tile);
    return (n + tile - 1) / tile;
}

// ot_spread without any allocation (work given, or ATOMIC).
int spread_noalloc(const ot_tree *t, const void *force, const void *pos, const int32_t *ids, int32_t dtype, int64_t n,
                   int32_t mode, int32_t accumulate, void *field_out, void *work, void *stream)
{
    return run_pass(t, kOpSpread, nullptr, force, pos, dtype, n, mode, accumulate, nullptr, nullptr, field_out,
                    nullptr, ids, work, (hipStream_t)stream, false);
}

}  // namespace ot

using namespace ot;

extern "C" int64_t ot_spread_workspace_bytes(const ot_tree *t)
{
    return t ? spread_ws_bytes(t->n_leaves) : 0;
}

extern "C" int ot_locate(const ot_tree *t, const void *pos, int32_t dtype, int64_t n, int32_t *ids, void *stream)
{
    return run_pass(t, kOpLocate, nullptr, nullptr, pos, dtype, n, OT_SPREAD_ATOMIC, 0, ids, nullptr, nullptr, nullptr,
                    nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int ot_interpolate(const ot_tree *t, const void *field, const void *pos, const int32_t *ids,
                              int32_t dtype, int64_t n, void *vel, void *stream)
{
    return run_pass(t, kOpInterp, field, nullptr, pos, dtype, n, OT_SPREAD_ATOMIC, 0, nullptr, vel, nullptr, nullptr,
                    ids, nullptr, (hipStream_t)stream);
}

extern "C" int ot_spread(const ot_tree *t, const void *force, const void *pos, const int32_t *ids, int32_t dtype,
                         int64_t n, int32_t mode, int32_t accumulate, void *field_out, void *work, void *stream)
{
    return run_pass(t, kOpSpread, nullptr, force, pos, dtype, n, mode, accumulate, nullptr, nullptr, field_out,
                    nullptr, ids, work, (hipStream_t)stream);
}

extern "C" int ot_track(const ot_tree *t, int32_t ops, const void *field, const void *force, const void *pos,
                        int32_t dtype, int64_t n, int32_t mode, int32_t accumulate, int32_t *ids, void *vel,
                        void *field_out, void *work, void *stream)
{
    if (ops <= 0 || ops > 7) return fail(OT_ERR_INVALID, "ops must be a non-empty combination of OT_OP_* bits");
    return run_pass(t, ops, field, force, pos, dtype, n, mode, accumulate, ids, vel, field_out, nullptr, nullptr, work,
                    (hipStream_t)stream);
}

extern "C" int ot_grad_pos(const ot_tree *t, const void *field, const void *vec, const void *pos, const int32_t *ids,
                           int32_t dtype, int64_t n, void *grad, void *stream)
{
    return run_pass(t, kOpGrad, field, vec, pos, dtype, n, OT_SPREAD_ATOMIC, 0, nullptr, nullptr, nullptr, grad, ids,
                    nullptr, (hipStream_t)stream);
}

extern "C" int ot_interp_grad_pos(const ot_tree *t, const void *field, const void *grad_vel, const void *pos,
                                  const int32_t *ids, int32_t dtype, int64_t n, void *grad_pos, void *stream)
{
    return ot_grad_pos(t, field, grad_vel, pos, ids, dtype, n, grad_pos, stream);
}

extern "C" int ot_spread_grad_pos(const ot_tree *t, const void *grad_field, const void *force, const void *pos,
                                  const int32_t *ids, int32_t dtype, int64_t n, void *grad_pos, void *stream)
{
    return ot_grad_pos(t, grad_field, force, pos, ids, dtype, n, grad_pos, stream);
}

extern "C" int ot_interp_backward(const ot_tree *t, const void *field, const void *grad_vel, const void *pos,
                                  const int32_t *ids, int32_t dtype, int64_t n, int32_t mode, int32_t accumulate,
                                  void *grad_field, void *grad_pos, void *work, void *stream)
{
    int ops = (grad_field ? (int)kOpSpread : 0) | (grad_pos ? (int)kOpGrad : 0);
    if (n == 0) ops &= ~(int)kOpGrad;   // no points: no position gradient (grad_field is still cleared)
    if (!ops) {
        if (n == 0) return check_common(t, dtype, n, pos);
        return fail(OT_ERR_INVALID, "ot_interp_backward: both outputs are NULL");
    }
    return run_pass(t, ops, field, grad_vel, pos, dtype, n, mode, accumulate, nullptr, nullptr, grad_field, grad_pos,
                    ids, work, (hipStream_t)stream);
}

extern "C" int ot_spread_backward(const ot_tree *t, const void *grad_field, const void *force, const void *pos,
                                  const int32_t *ids, int32_t dtype, int64_t n, void *grad_force, void *grad_pos,
                                  void *stream)
{
    const int ops = (grad_force ? (int)kOpInterp : 0) | (grad_pos ? (int)kOpGrad : 0);
    if (n == 0) return check_common(t, dtype, n, pos);   // both outputs are per point: nothing to do
    if (!ops) return fail(OT_ERR_INVALID, "ot_spread_backward: both outputs are NULL");
    return run_pass(t, ops, grad_field, force, pos, dtype, n, OT_SPREAD_ATOMIC, 0, nullptr, grad_force, nullptr,
                    grad_pos, ids, nullptr, (hipStream_t)stream);
}
