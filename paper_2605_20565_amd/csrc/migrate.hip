// Phase I of the migration of Lagrangian points (Algorithm 2) on one device.
//
// relocate: the host of every moved point and the number of points whose
// host changed (the leavers of phase I).  The paper checks the previous host
// first because its search is a binary search; here a fresh descent is one
// or two loads from the (cached) descent table, cheaper than fetching the
// previous leaf's key and level, so every point descends and is compared
// with its previous id.
// find_owner: under a partition of the leaves into contiguous Morton ranges
// (Sec. 3.1), the owner of a point is the range holding the Morton key of
// its finest-level cell, found by a binary search over the P + 1 splitters;
// the per-owner counts are the sizes of the send buffers of phase II.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ot_common.h"
#include "track_device.h"

namespace ot {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxOwners = 4096;

template <int THREADS>
__device__ __forceinline__ void block_count_to(unsigned long long v, unsigned long long *sh, unsigned long long *out)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += (unsigned long long)__shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < THREADS / 64; ++w) v += sh[w];
        if (v) atomicAdd(out, v);
    }
}

// Cells of a thread's ITEMS points of one tile (ITEMS * THREADS points from
// base), all loaded before any is used, at clamped indices.
template <typename T, int ITEMS, int THREADS>
__device__ __forceinline__ void tile_cells(const TreeView &tv, const T *__restrict__ pos, int64_t n, int64_t base,
                                           uint32_t (&I)[ITEMS][3], bool (&ok)[ITEMS])
{
    T X[ITEMS][3];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t k = base + j * THREADS + threadIdx.x;
        const int64_t kc = k < n ? k : n - 1;
#pragma unroll
        for (int d = 0; d < 3; ++d) X[j][d] = pos[3 * kc + d];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) ok[j] = point_cell<T>(tv, X[j][0], X[j][1], X[j][2], I[j]);
}

// Bound by memory (20 bytes a point in FP32).  A workgroup walks over tiles of
// ITEMS points per thread whose table loads are in flight together, and adds
// its count of moved points once: one add per 256 points had put 39,000 adds
// on one address (10 ns each on this target) and the kernel at 478 us for 10^7
// points; it takes 79 now.
template <typename T, int ITEMS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_relocate(TreeView tv, const T *__restrict__ pos, int64_t n,
                                                       int32_t *__restrict__ ids,
                                                       unsigned long long *__restrict__ moved)
{
    __shared__ unsigned long long sh[THREADS / 64];
    const int rsh = tv.L - tv.lev[0];
    unsigned long long changed = 0;
    for (int64_t base = blockIdx.x * (int64_t)(THREADS * ITEMS); base < n;
         base += gridDim.x * (int64_t)(THREADS * ITEMS)) {
        uint32_t I[ITEMS][3], root[ITEMS], e[ITEMS];
        int32_t prev[ITEMS];
        bool ok[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t k = base + j * THREADS + threadIdx.x;
            prev[j] = ids[k < n ? k : n - 1];
        }
        tile_cells<T, ITEMS, THREADS>(tv, pos, n, base, I, ok);
        // root summary, the root where it has no answer, then deeper levels
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            root[j] = interleave3(I[j][0] >> rsh, I[j][1] >> rsh, I[j][2] >> rsh);
            e[j] = tv.summary ? ld_summary(tv, root[j] >> 3) : kSplit;
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (!(e[j] & kSplit)) e[j] += root[j] & 7u;
            else e[j] = descend_below_root(tv, ld_table(tv, root[j]), I[j][0], I[j][1], I[j][2]);
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t k = base + j * THREADS + threadIdx.x;
            const int32_t id = ok[j] ? (int32_t)(e[j] & kIdMask) : -1;
            if (k < n) {
                ids[k] = id;
                changed += id != prev[j] ? 1ull : 0ull;
            }
        }
    }
    if (moved) block_count_to<THREADS>(changed, sh, moved);
}

__global__ void k_leaf_splitters(const uint64_t *__restrict__ keys, int64_t n_leaves, int P, int L,
                                 int64_t *__restrict__ split)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r > P) return;
    if (r == 0) split[0] = 0;
    else if (r == P) split[P] = (int64_t)1 << (3 * L);
    else split[r] = (int64_t)keys[((int64_t)r * n_leaves) / P];
}

// Splitters staged in LDS.  A workgroup walks over tiles of ITEMS points per
// thread, loaded together (one after another they had taken 112 us for 10^7
// points and 8 owners), and adds its counts to device memory once.  LDS is
// sized by the owners: at 48 KB for the most there can be, three of a CU's four
// workgroups fitted, and the last quarter of the walkers ran alone (80 us).
// Counts: for up to kBallotOwners owners every wave counts each owner with
// one ballot (no same-address atomics), else LDS atomics.
constexpr int kBallotOwners = 32;

template <typename T, int ITEMS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_find_owner(TreeView tv, const int64_t *__restrict__ split, int P,
                                                         const T *__restrict__ pos, int64_t n,
                                                         int32_t *__restrict__ owner,
                                                         unsigned long long *__restrict__ counts)
{
    extern __shared__ int64_t s_split[];   // P + 1 splitters, then P counts
    unsigned int *hist = reinterpret_cast<unsigned int *>(s_split + P + 1);
    for (int i = threadIdx.x; i <= P; i += THREADS) s_split[i] = split[i];
    for (int i = threadIdx.x; i < P; i += THREADS) hist[i] = 0u;
    __syncthreads();
    for (int64_t base = blockIdx.x * (int64_t)(THREADS * ITEMS); base < n;
         base += gridDim.x * (int64_t)(THREADS * ITEMS)) {
        uint32_t I[ITEMS][3];
        bool ok[ITEMS];
        int32_t o[ITEMS];
        tile_cells<T, ITEMS, THREADS>(tv, pos, n, base, I, ok);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t k = base + j * THREADS + threadIdx.x;
            const int64_t key = (int64_t)(split3_21(I[j][0]) | (split3_21(I[j][1]) << 1) | (split3_21(I[j][2]) << 2));
            // largest r in [0, P) with split[r] <= key
            int lo = 0, hi = P;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_split[mid] <= key) lo = mid;
                else hi = mid;
            }
            o[j] = k < n && ok[j] ? lo : -1;
            if (k < n) owner[k] = o[j];
        }
        if (counts) {
            if (P <= kBallotOwners) {
                for (int r = 0; r < P; ++r) {
                    unsigned c = 0u;
#pragma unroll
                    for (int j = 0; j < ITEMS; ++j) c += (unsigned)__popcll(__ballot(o[j] == r));
                    if ((threadIdx.x & 63) == 0 && c) atomicAdd(&hist[r], c);
                }
            } else {
#pragma unroll
                for (int j = 0; j < ITEMS; ++j)
                    if (o[j] >= 0) atomicAdd(&hist[o[j]], 1u);
            }
        }
    }
    if (counts) {
        __syncthreads();
        for (int i = threadIdx.x; i < P; i += THREADS)
            if (hist[i]) atomicAdd(&counts[i], (unsigned long long)hist[i]);
    }
}

// Launch of the two kernels above: kWide points per thread once that still
// gives every CU a workgroup.  find_owner's workgroups end in an add per owner
// to the same few words, so its large calls take few of them, of kManyThreads
// threads: 10^7 points and 8 owners 52 us, and 57 in workgroups of 256 (64
// owners 53 and 63).  Relocation, with one add each, takes 79 us either way,
// and with 2, 4 or 8 points per thread.
constexpr int kWide = 4, kWalkers = 1024;
constexpr int kManyThreads = 1024, kManyWalkers = 512;

unsigned walkers(int64_t n, int64_t per) { return (unsigned)std::min<int64_t>((n + per - 1) / per, kWalkers); }

template <typename T>
void relocate(const TreeView &tv, const T *pos, int64_t n, int32_t *ids, unsigned long long *moved, hipStream_t s)
{
    if (n >= (int64_t)kThreads * kWide * 256)
        hipLaunchKernelGGL((k_relocate<T, kWide, kThreads>), dim3(walkers(n, kThreads * kWide)), dim3(kThreads), 0, s,
                           tv, pos, n, ids, moved);
    else
        hipLaunchKernelGGL((k_relocate<T, 1, kThreads>), dim3(walkers(n, kThreads)), dim3(kThreads), 0, s, tv, pos, n,
                           ids, moved);
}

template <typename T>
void find_owner(const TreeView &tv, const int64_t *split, int P, const T *pos, int64_t n, int32_t *owner,
                unsigned long long *counts, hipStream_t s)
{
    const size_t lds = sizeof(int64_t) * ((size_t)P + 1) + sizeof(unsigned) * (size_t)P;   // 48 KB at most
    if (n >= (int64_t)kManyThreads * kWide * 256)
        hipLaunchKernelGGL((k_find_owner<T, kWide, kManyThreads>), dim3(kManyWalkers), dim3(kManyThreads), lds, s, tv,
                           split, P, pos, n, owner, counts);
    else if (n >= (int64_t)kThreads * kWide * 256)
        hipLaunchKernelGGL((k_find_owner<T, kWide, kThreads>), dim3(walkers(n, kThreads * kWide)), dim3(kThreads), lds,
                           s, tv, split, P, pos, n, owner, counts);
    else
        hipLaunchKernelGGL((k_find_owner<T, 1, kThreads>), dim3(walkers(n, kThreads)), dim3(kThreads), lds, s, tv, split,
                           P, pos, n, owner, counts);
}

}  // namespace
}  // namespace ot

using namespace ot;

extern "C" int ot_relocate(const ot_tree *t, const void *pos, int32_t dtype, int64_t n, int32_t *ids, int64_t *moved,
                           void *stream)
{
    if (!t) return fail(OT_ERR_INVALID, "ot_relocate: tree is NULL");
    if (dtype != OT_F32 && dtype != OT_F64) return fail(OT_ERR_INVALID, "dtype must be OT_F32 or OT_F64");
    if (n < 0) return fail(OT_ERR_INVALID, "n < 0");
    if (n > 0 && (!pos || !ids)) return fail(OT_ERR_INVALID, "ot_relocate: pos or ids is NULL");
    hipStream_t s = (hipStream_t)stream;
    unsigned long long *mv = (unsigned long long *)moved;
    if (mv) hipLaunchKernelGGL(k_fill<unsigned long long>, dim3(1), dim3(64), 0, s, mv, (int64_t)1, 0ull);
    if (n > 0) {
        if (dtype == OT_F32) relocate<float>(t->view, (const float *)pos, n, ids, mv, s);
        else relocate<double>(t->view, (const double *)pos, n, ids, mv, s);
    }
    OT_HIP(hipGetLastError());
    return OT_OK;
}

extern "C" int ot_leaf_splitters(const ot_tree *t, int32_t P, int64_t *splitters, void *stream)
{
    if (!t || !splitters) return fail(OT_ERR_INVALID, "ot_leaf_splitters: NULL argument");
    if (P < 1 || P > kMaxOwners || P > t->n_leaves) return fail(OT_ERR_INVALID, "ot_leaf_splitters: need 1 <= P <= min(4096, n_leaves)");
    hipLaunchKernelGGL(k_leaf_splitters, dim3((unsigned)((P + 1 + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       t->keys, t->n_leaves, (int)P, (int)t->l_max, splitters);
    OT_HIP(hipGetLastError());
    return OT_OK;
}

extern "C" int ot_find_owner(const int64_t *splitters, int32_t P, int32_t l_max, int32_t periodic, const void *pos,
                             int32_t dtype, int64_t n, int32_t *owner, int64_t *counts, void *stream)
{
    if (P < 1 || P > kMaxOwners) return fail(OT_ERR_INVALID, "ot_find_owner: need 1 <= P <= 4096");
    if (l_max < 0 || l_max > 21) return fail(OT_ERR_LEVEL_RANGE, "ot_find_owner: l_max outside [0, 21]");
    if (dtype != OT_F32 && dtype != OT_F64) return fail(OT_ERR_INVALID, "dtype must be OT_F32 or OT_F64");
    if (n < 0) return fail(OT_ERR_INVALID, "n < 0");
    if (!splitters || (n > 0 && (!pos || !owner))) return fail(OT_ERR_INVALID, "ot_find_owner: NULL array");
    hipStream_t s = (hipStream_t)stream;
    unsigned long long *cnt = (unsigned long long *)counts;
    if (cnt) hipLaunchKernelGGL(k_fill<unsigned long long>, dim3(16), dim3(256), 0, s, cnt, (int64_t)P, 0ull);
    TreeView tv{};
    tv.L = l_max;
    tv.periodic = periodic ? 1 : 0;
    if (n > 0) {
        if (dtype == OT_F32) find_owner<float>(tv, splitters, (int)P, (const float *)pos, n, owner, cnt, s);
        else find_owner<double>(tv, splitters, (int)P, (const double *)pos, n, owner, cnt, s);
    }
    OT_HIP(hipGetLastError());
    return OT_OK;
}
