// Tree construction on the GPU: Morton keys of leaf anchors, an LSD radix
// sort of the keys staged in LDS, validation that the sorted leaves tile the
// unit cube, and the descent table used by every lookup.
//
// Sec. 3.1 of the paper keeps the leaves of each tree in an array sorted by
// Morton (Z-order) index; Algorithm 1 binary-searches that array once per
// level.  Here the sorted array is built once per tree and indexed by a radix
// table over groups of three Morton digits, so a lookup is one dependent
// load per three levels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "memory.h"
#include "ot_common.h"

namespace ot {

namespace {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;   // 2048 keys per workgroup
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;

__global__ void k_encode_keys(const uint32_t *__restrict__ a, int64_t n, uint64_t *__restrict__ keys)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    // Anchors at or above 2^21 keep their high bits so that validation sees them.
    uint64_t x = a[3 * i], y = a[3 * i + 1], z = a[3 * i + 2];
    uint64_t k = split3_21(x) | (split3_21(y) << 1) | (split3_21(z) << 2);
    if ((x | y | z) >> 21) k |= 0x8000000000000000ull;
    keys[i] = k;
}

// -- block-wide exclusive scan over 256 threads (4 waves of 64) -------------
__device__ __forceinline__ uint32_t block_exscan_256(uint32_t v, uint32_t *sh_w, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) sh_w[wid] = x;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSortThreads / 64; ++w) {
        uint32_t s = sh_w[w];
        if (w < wid) pre += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return pre + x - v;
}

}  // namespace

// -- device-wide exclusive scan of uint32 (reduce/scan per 2048 + recursion) -
__global__ __launch_bounds__(kSortThreads) void k_scan_tiles(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                                                             int64_t n, uint32_t *__restrict__ sums)
{
    __shared__ uint32_t sh_w[kSortThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kSortTile + (int64_t)threadIdx.x * kSortItems;
    uint32_t v[kSortItems], s = 0;
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        v[j] = (base + j < n) ? in[base + j] : 0u;
        s += v[j];
    }
    uint32_t tot;
    uint32_t pre = block_exscan_256(s, sh_w, tot);
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        if (base + j < n) out[base + j] = pre;
        pre += v[j];
    }
    if (threadIdx.x == 0 && sums) sums[blockIdx.x] = tot;
}

__global__ void k_scan_add(uint32_t *__restrict__ out, int64_t n, const uint32_t *__restrict__ offs)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] += offs[i / kSortTile];
}

// Exclusive scan of n uint32 values (n < 2^32 total).  tmp must hold
// scan_tmp_words(n) words.
int64_t scan_tmp_words(int64_t n)
{
    int64_t w = 0;
    while (n > kSortTile) {
        n = (n + kSortTile - 1) / kSortTile;
        w += 2 * n;
    }
    return w + 1;
}

void exclusive_scan(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s)
{
    if (n <= 0) return;
    int64_t nb = (n + kSortTile - 1) / kSortTile;
    if (nb == 1) {
        hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(kSortThreads), 0, s, in, out, n, (uint32_t *)nullptr);
        return;
    }
    uint32_t *sums = tmp, *sums_scan = tmp + nb;
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nb), dim3(kSortThreads), 0, s, in, out, n, sums);
    exclusive_scan(sums, sums_scan, nb, tmp + 2 * nb, s);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, n, sums_scan);
}

const uint32_t *exclusive_scan_split(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp, hipStream_t s)
{
    static_assert(kScanBlock == kSortTile, "the split scan's block is the scan tile");
    const int64_t nb = (n + kSortTile - 1) / kSortTile;
    if (nb <= 1 || nb > kSortTile) {
        exclusive_scan(in, out, n, tmp, s);
        return nullptr;
    }
    uint32_t *sums = tmp, *sums_scan = tmp + nb;
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nb), dim3(kSortThreads), 0, s, in, out, n, sums);
    hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(kSortThreads), 0, s, sums, sums_scan, nb, (uint32_t *)nullptr);
    return sums_scan;
}

// -- stable LSD radix sort of uint32 or uint64 keys with their input positions --
// Tile of workgroup blockIdx.x: each of the 8 XCDs takes a contiguous range of
// tiles, so that the ends of neighbouring tiles' runs of one digit meet in one
// L2.
__device__ __forceinline__ int xcd_tile(int nblocks)
{
    const int xg = (int)(blockIdx.x & 7u), xk = (int)(blockIdx.x >> 3), xq = nblocks >> 3, xr = nblocks & 7;
    return xg * xq + (xg < xr ? xg : xr) + xk;
}

// LDS index with one pad word per 32: reads of kSortItems words in a row and
// striped ones both spread over the banks.
__device__ __forceinline__ int sort_pad(int i) { return i + (i >> 5); }
constexpr int kSortPadded = kSortTile + kSortTile / 32;

template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const K *__restrict__ keys, int64_t n, int shift,
                                                             uint32_t dmask, uint32_t *__restrict__ counts, int nblocks)
{
    __shared__ uint32_t hist[kRadix];
    for (int i = threadIdx.x; i < kRadix; i += kSortThreads) hist[i] = 0;
    __syncthreads();
    const int tile = xcd_tile(nblocks);
    const int64_t base = (int64_t)tile * kSortTile;
    // all of a thread's keys loaded (clamped) before any is counted
    K k[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int64_t i = base + j * kSortThreads + threadIdx.x;
        k[j] = keys[i < n ? i : base];
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (base + j * kSortThreads + threadIdx.x < n) atomicAdd(&hist[(uint32_t)(k[j] >> shift) & dmask], 1u);
    __syncthreads();
    for (int d = threadIdx.x; d <= (int)dmask; d += kSortThreads) counts[(int64_t)d * nblocks + tile] = hist[d];
}

// Stable scatter of one tile: words of digit and place in the tile are sorted
// by the digit with one-bit splits in LDS, then every key goes to
// offset[digit][tile] + (its rank among the tile's keys with that digit).
// Keys and values are loaded in input order and stored in sorted order, both
// coalesced, and pass LDS once each.  vin = NULL: the first pass, whose values
// are the input positions.
// Bound by the split rounds' LDS traffic and by the runs' partial lines, not by
// bytes: 10^7 32-bit keys take 63 us a pass (160 MB, 2.5 TB/s), where moving
// whole 12-byte pairs through every split, blocked loads and stores and a
// serial scan of the 256 digits had taken 264.
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const K *__restrict__ kin, const int32_t *__restrict__ vin, K *__restrict__ kout,
    int32_t *__restrict__ vout, int64_t n, int shift, int pbits, const uint32_t *__restrict__ offs,
    const uint32_t *__restrict__ offs_hi, int nblocks)
{
    static_assert(kSortTile <= 1 << 16 && kRadixBits <= 16, "digit and place share a word");
    __shared__ uint32_t sw[kSortPadded];
    __shared__ K stg[kSortPadded];
    __shared__ uint32_t sh_w[kSortThreads / 64];
    __shared__ uint32_t dstart[kRadix];
    __shared__ uint32_t dcount[kRadix];

    const uint32_t dmask = (1u << pbits) - 1u;
    const int tile = xcd_tile(nblocks);
    const int64_t base = (int64_t)tile * kSortTile;
    const int64_t rem = n - base;
    const int valid = rem < kSortTile ? (int)rem : kSortTile;
    // loads at clamped places (the tile's first key stands in for the padding)
    K k[kSortItems];
    int32_t v[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int li = j * kSortThreads + threadIdx.x;
        k[j] = kin[base + (li < valid ? li : 0)];
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int li = j * kSortThreads + threadIdx.x;
        v[j] = vin ? vin[base + (li < valid ? li : 0)] : (int32_t)(base + li);
    }
    dcount[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int li = j * kSortThreads + threadIdx.x;
        // the padding has the largest digit and the last places: it stays behind
        const uint32_t d = li < valid ? (uint32_t)(k[j] >> shift) & dmask : dmask;
        if (li < valid) atomicAdd(&dcount[d], 1u);
        sw[sort_pad(li)] = d << 16 | (uint32_t)li;
        stg[sort_pad(li)] = k[j];
    }
    __syncthreads();
    uint32_t tot;
    dstart[threadIdx.x] = block_exscan_256(dcount[threadIdx.x], sh_w, tot);
    const int t0 = threadIdx.x * kSortItems;
    uint32_t x[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) x[j] = sw[sort_pad(t0 + j)];
    for (int b = 0; b < pbits; ++b) {
        uint32_t zeros = 0;
#pragma unroll
        for (int j = 0; j < kSortItems; ++j) zeros += 1u - ((x[j] >> (16 + b)) & 1u);
        uint32_t total_zeros;
        uint32_t zb = block_exscan_256(zeros, sh_w, total_zeros);   // every thread has read its words
#pragma unroll
        for (int j = 0; j < kSortItems; ++j) {
            const uint32_t bit = (x[j] >> (16 + b)) & 1u;
            const uint32_t g = (uint32_t)(t0 + j);
            const uint32_t pos = bit ? total_zeros + (g - zb) : zb;
            zb += 1u - bit;
            sw[sort_pad((int)pos)] = x[j];
        }
        __syncthreads();
        if (b + 1 < pbits) {
#pragma unroll
            for (int j = 0; j < kSortItems; ++j) x[j] = sw[sort_pad(t0 + j)];
        }
    }
    int64_t dst[kSortItems];
    int src[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int i = j * kSortThreads + threadIdx.x;
        const uint32_t w = sw[sort_pad(i)], d = w >> 16;
        const int64_t oi = (int64_t)d * nblocks + tile;
        const int64_t o = (int64_t)offs[oi] + (offs_hi ? (int64_t)offs_hi[oi / kScanBlock] : 0);
        dst[j] = i < valid ? o + (i - (int)dstart[d]) : -1;
        src[j] = sort_pad((int)(w & 0xFFFFu));
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const K key = stg[src[j]];
        if (dst[j] >= 0) kout[dst[j]] = key;
    }
    __syncthreads();   // the keys are read
    uint32_t *sv = reinterpret_cast<uint32_t *>(stg);
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) sv[sort_pad(j * kSortThreads + threadIdx.x)] = (uint32_t)v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int32_t val = (int32_t)sv[src[j]];
        if (dst[j] >= 0) vout[dst[j]] = val;
    }
}

namespace {

template <typename K>
__global__ void k_copy_iota(const K *__restrict__ kin, K *__restrict__ k, int32_t *__restrict__ v, int64_t n)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    k[i] = kin[i];
    v[i] = (int32_t)i;
}

__global__ void k_gather_levels(const uint8_t *__restrict__ lin, const int32_t *__restrict__ perm,
                                uint8_t *__restrict__ lout, int64_t n)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) lout[i] = lin[perm[i]];
}

// -- validation: the sorted leaves tile the cube exactly --------------------
enum : unsigned { kErrPartition = 1u, kErrDup = 2u, kErrLevel = 4u };

__global__ void k_validate(const uint64_t *__restrict__ keys, const uint8_t *__restrict__ lv, int64_t n,
                           int l_min, int L, unsigned *__restrict__ err)
{
    int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    unsigned e = 0;
    const uint64_t k = keys[j];
    const int l = lv[j];
    if (l < l_min || l > L || (k >> (3 * L)) != 0) {
        e |= kErrLevel;
    } else {
        const uint64_t vol = 1ull << (3 * (L - l));
        if (k & (vol - 1)) e |= kErrPartition;
        if (j == 0 && k != 0) e |= kErrPartition;
        if (j + 1 < n) {
            const uint64_t kn = keys[j + 1];
            if (kn == k) e |= kErrDup;
            else if (k + vol != kn) e |= kErrPartition;
        } else if (k + vol != (1ull << (3 * L))) {
            e |= kErrPartition;
        }
    }
    if (e) atomicOr(err, e);
}

// -- descent table ------------------------------------------------------------
// Number of split cells at each table level t (cells of level lev[t] covered
// by finer leaves): counted at the first leaf inside each such cell.  Few
// workgroups: each ends in an atomic per level on the same words.
__global__ void k_count_splits(const uint64_t *__restrict__ keys, const uint8_t *__restrict__ lv, int64_t n,
                               TreeView tv, unsigned long long *__restrict__ counts)
{
    __shared__ unsigned sc[kMaxTabLevels];
    if (threadIdx.x < kMaxTabLevels) sc[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[j];
        const int l = lv[j];
        for (int t = 0; t + 1 < tv.nlev; ++t) {
            const uint64_t cell = 1ull << (3 * (tv.L - tv.lev[t]));
            if (l > tv.lev[t] && (k & (cell - 1)) == 0) atomicAdd(&sc[t], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < kMaxTabLevels && sc[threadIdx.x]) atomicAdd(&counts[threadIdx.x], (unsigned long long)sc[threadIdx.x]);
}

__global__ void k_split_flags(const uint64_t *__restrict__ keys, const uint8_t *__restrict__ lv, int64_t n, int L,
                              int lev_t, uint32_t *__restrict__ flags)
{
    int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    const uint64_t cell = 1ull << (3 * (L - lev_t));
    flags[j] = (lv[j] > lev_t && (keys[j] & (cell - 1)) == 0) ? 1u : 0u;
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Write the entries of table level t.  Leaves with lev[t-1] < level <= lev[t]
// fill the 8^(lev[t]-level) entries they cover; the first leaf of each split
// level-lev[t] cell writes the pointer to its sub-table and the sub-table's
// anchor (anchors: of the next table level).
__global__ void k_write_level(const uint64_t *__restrict__ keys, const uint8_t *__restrict__ lv, int64_t n,
                              TreeView tv, uint32_t *__restrict__ table, int t, const uint32_t *__restrict__ sub_ids,
                              uint64_t *__restrict__ anchors)
{
    int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int l = lv[j];
    if (t > 0 && l <= tv.lev[t - 1]) return;
    const uint64_t k = keys[j];
    const uint32_t ax = compact3_21(k), ay = compact3_21(k >> 1), az = compact3_21(k >> 2);
    const int L = tv.L;
    int64_t base;
    uint32_t digit;
    if (t == 0) {
        const int s = L - tv.lev[0];
        base = 0;
        digit = interleave3(ax >> s, ay >> s, az >> s);
    } else {
        // walk the already written levels 0..t-1; the leaf lies in a split cell at each
        const int s0 = L - tv.lev[0];
        uint32_t e = table[interleave3(ax >> s0, ay >> s0, az >> s0)];
        for (int u = 1; u < t; ++u) {
            const int d = tv.lev[u] - tv.lev[u - 1];
            const int s = L - tv.lev[u];
            const uint32_t m = (1u << d) - 1u;
            e = table[tv.off[u] + (int64_t)(e & ~kSplit) * (int64_t(1) << (3 * d)) +
                      interleave3((ax >> s) & m, (ay >> s) & m, (az >> s) & m)];
        }
        const int d = tv.lev[t] - tv.lev[t - 1];
        const int s = L - tv.lev[t];
        const uint32_t m = (1u << d) - 1u;
        base = tv.off[t] + (int64_t)(e & ~kSplit) * (int64_t(1) << (3 * d));
        digit = interleave3((ax >> s) & m, (ay >> s) & m, (az >> s) & m);
    }
    if (l <= tv.lev[t]) {
        const uint32_t ent = ((uint32_t)l << kLevelShift) | (uint32_t)j;
        const int64_t cnt = int64_t(1) << (3 * (tv.lev[t] - l));
        for (int64_t c = 0; c < cnt; ++c) table[base + digit + c] = ent;
    } else {
        const uint64_t cell = 1ull << (3 * (L - tv.lev[t]));
        if ((k & (cell - 1)) == 0) {
            table[base + digit] = kSplit | sub_ids[j];
            anchors[sub_ids[j]] = k;
        }
    }
}

// Summary of the root one level up: entry m describes the 8 root cells of
// the level-(r-1) cell m.  When all 8 are leaves of level r, they are 8
// consecutive leaves in Z-order and the entry is the first one's (so the
// leaf of child c is entry + c); otherwise it is kSplit.
__global__ void k_root_summary(const uint32_t *__restrict__ root, int64_t m_cells, int r, uint32_t *__restrict__ sum)
{
    const int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (m >= m_cells) return;
    bool uniform = true;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const uint32_t e = root[8 * m + c];
        uniform = uniform && !(e & kSplit) && (int)((e >> kLevelShift) & 31u) == r;
    }
    sum[m] = uniform ? root[8 * m] : kSplit;
}

__global__ void k_count_value(const uint32_t *__restrict__ p, int64_t n, uint32_t v, unsigned *__restrict__ out)
{
    unsigned c = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        c += (p[i] == v);
    if (c) atomicAdd(out, c);
}

inline unsigned nblk(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// A build's block: given back at the end, when the build's work on it is done.
struct BuildBlock {
    Block b;
    hipStream_t s;
    explicit BuildBlock(hipStream_t st) : s(st) {}
    BuildBlock(const BuildBlock &) = delete;
    BuildBlock &operator=(const BuildBlock &) = delete;
    ~BuildBlock()
    {
        if (!b.p) return;
        if (hipStreamSynchronize(s) == hipSuccess) block_give(b);
        else (void)hipFree(b.p);
    }
    int take(size_t bytes)
    {
        b = block_take(bytes);
        if (b.p) return OT_OK;
        return fail(OT_ERR_OOM, "device allocation of " + std::to_string(bytes) + " bytes failed");
    }
    Block release()
    {
        const Block r = b;
        b.p = nullptr;
        return r;
    }
};

size_t align256(int64_t b) { return (size_t)((b + 255) & ~int64_t(255)); }

}  // namespace

// Device workspace (bytes) of radix_sort_pairs for n keys.
int64_t radix_ws_bytes(int64_t n)
{
    const int64_t nb = (n + kSortTile - 1) / kSortTile;
    const int64_t nc = (int64_t)kRadix * nb;
    return 4 * (2 * nc + scan_tmp_words(nc)) + 256;
}

// Stable LSD radix sort of the keys kin over their low `bits` bits, values
// being the input positions, without allocating (ws: radix_ws_bytes(n) bytes).
// Passes write (ka, va) and (kb, vb) in turn, the first (ka, va); kin may be kb.
// *k_res / *v_res point at the result; with no bits to sort the keys are copied
// to (ka, va).
template <typename K>
void radix_sort_pairs(const K *kin, K *ka, int32_t *va, K *kb, int32_t *vb, int64_t n, int bits, void *ws, K **k_res,
                      int32_t **v_res, hipStream_t s)
{
    *k_res = ka;
    *v_res = va;
    if (n <= 0) return;
    if (bits <= 0) {
        hipLaunchKernelGGL(k_copy_iota<K>, dim3(nblk(n)), dim3(256), 0, s, kin, ka, va, n);
        return;
    }
    // the passes share the bits evenly: fewer split rounds, longer runs
    const int passes = (bits + kRadixBits - 1) / kRadixBits, pbits = (bits + passes - 1) / passes;
    const uint32_t dmask = (1u << pbits) - 1u;
    const int nb = (int)((n + kSortTile - 1) / kSortTile);
    const int64_t ncounts = (int64_t)(dmask + 1) * nb;
    uint32_t *counts = (uint32_t *)ws, *offs = counts + ncounts, *tmp = offs + ncounts;
    const int32_t *vin = nullptr;
    for (int p = 0; p < passes; ++p) {
        hipLaunchKernelGGL(k_radix_hist<K>, dim3(nb), dim3(kSortThreads), 0, s, kin, n, p * pbits, dmask, counts, nb);
        const uint32_t *offs_hi = exclusive_scan_split(counts, offs, ncounts, tmp, s);
        hipLaunchKernelGGL(k_radix_scatter<K>, dim3(nb), dim3(kSortThreads), 0, s, kin, vin, ka, va, n, p * pbits, pbits,
                           (const uint32_t *)offs, offs_hi, nb);
        *k_res = ka;
        *v_res = va;
        kin = ka;
        vin = va;
        std::swap(ka, kb);
        std::swap(va, vb);
    }
}
template void radix_sort_pairs<uint32_t>(const uint32_t *, uint32_t *, int32_t *, uint32_t *, int32_t *, int64_t, int,
                                         void *, uint32_t **, int32_t **, hipStream_t);
template void radix_sort_pairs<uint64_t>(const uint64_t *, uint64_t *, int32_t *, uint64_t *, int32_t *, int64_t, int,
                                         void *, uint64_t **, int32_t **, hipStream_t);

}  // namespace ot

using namespace ot;

extern "C" int ot_encode_keys(const uint32_t *anchors, int64_t n, int32_t l_max, uint64_t *keys, void *stream)
{
    if (n < 0 || (n > 0 && (!anchors || !keys))) return fail(OT_ERR_INVALID, "ot_encode_keys: bad arguments");
    if (l_max < 0 || l_max > 21) return fail(OT_ERR_LEVEL_RANGE, "ot_encode_keys: l_max must be in [0, 21]");
    if (n == 0) return OT_OK;
    hipLaunchKernelGGL(k_encode_keys, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, anchors, n, keys);
    OT_HIP(hipGetLastError());
    return OT_OK;
}

extern "C" int ot_build_tree(const uint64_t *keys, const uint8_t *levels, int64_t n, const ot_tree_desc *desc,
                             int32_t *perm_out, void *stream, ot_tree **out)
{
    if (!out) return fail(OT_ERR_INVALID, "ot_build_tree: out is NULL");
    *out = nullptr;
    if (!desc || !keys || !levels || n <= 0) return fail(OT_ERR_INVALID, "ot_build_tree: bad arguments");
    const int L = desc->l_max, l_min = desc->l_min;
    if (L < 0 || L > 21 || l_min < 0 || l_min > L)
        return fail(OT_ERR_LEVEL_RANGE, "ot_build_tree: need 0 <= l_min <= l_max <= 21");
    if (n > kMaxLeaves) return fail(OT_ERR_CAPACITY, "ot_build_tree: more than 2^26 leaves");
    hipStream_t s = (hipStream_t)stream;
    int rc;

    // the tree's own block: sorted keys and levels; the build's: the other key
    // buffer (later the split flags and ids), two position buffers and scratch
    BuildBlock own(s), tmp(s);
    const size_t nk = align256(8 * n), nv = align256(4 * n);
    if ((rc = own.take(nk + align256(n))) ||
        (rc = tmp.take(2 * nv + 2 * nv + align256(radix_ws_bytes(n)) + align256(4 * scan_tmp_words(n)) + 256)))
        return rc;
    uint64_t *keys_own = (uint64_t *)own.b.p;
    uint8_t *lvs = (uint8_t *)own.b.p + nk;
    char *q = (char *)tmp.b.p;
    uint32_t *flags = (uint32_t *)q, *ids = (uint32_t *)(q + nv);
    uint64_t *keys_tmp = (uint64_t *)q;   // 8n bytes fit in 2 nv
    int32_t *va = (int32_t *)(q + 2 * nv), *vb = (int32_t *)(q + 3 * nv);
    void *sws = q + 4 * nv;
    uint32_t *stmp = (uint32_t *)((char *)sws + align256(radix_ws_bytes(n)));
    void *scratch = (char *)stmp + align256(4 * scan_tmp_words(n));
    // Keys of a valid tree use 3L bits; sort on those (others fail validation).
    // The last pass writes the tree's own buffer.
    const bool odd = ((3 * L + kRadixBits - 1) / kRadixBits) % 2 != 0 || L == 0;
    uint64_t *ks;
    int32_t *perm;
    radix_sort_pairs(keys, odd ? keys_own : keys_tmp, va, odd ? keys_tmp : keys_own, vb, n, 3 * L, sws, &ks, &perm, s);
    OT_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_gather_levels, dim3(nblk(n)), dim3(256), 0, s, levels, perm, lvs, n);

    // Table layout: root level r = min(l_min, 8), then steps of <= 3 levels.
    TreeView tv{};
    tv.L = L;
    tv.periodic = desc->periodic ? 1 : 0;
    tv.lev[0] = std::min(l_min, kMaxRootLevel);
    tv.nlev = 1;
    while (tv.lev[tv.nlev - 1] < L) {
        tv.lev[tv.nlev] = std::min(tv.lev[tv.nlev - 1] + 3, L);
        tv.nlev++;
    }

    unsigned *err = (unsigned *)scratch;
    unsigned long long *cnt = (unsigned long long *)((char *)scratch + 64);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t *)scratch, (int64_t)64, 0u);
    hipLaunchKernelGGL(k_validate, dim3(nblk(n)), dim3(256), 0, s, ks, (const uint8_t *)lvs, n, l_min, L, err);
    hipLaunchKernelGGL(k_count_splits, dim3(std::min(nblk(n), 512u)), dim3(256), 0, s, ks, (const uint8_t *)lvs, n, tv, cnt);
    OT_HIP(hipGetLastError());
    unsigned herr = 0;
    unsigned long long hcnt[kMaxTabLevels] = {0};
    OT_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, s));
    OT_HIP(hipMemcpyAsync(hcnt, cnt, sizeof(hcnt), hipMemcpyDeviceToHost, s));
    OT_HIP(hipStreamSynchronize(s));
    if (herr & kErrLevel) return fail(OT_ERR_LEVEL_RANGE, "ot_build_tree: leaf level outside [l_min, l_max] or key above 3*l_max bits");
    if (herr & kErrDup) return fail(OT_ERR_UNSORTED_DUP, "ot_build_tree: two leaves share a Morton key");
    if (herr & kErrPartition) return fail(OT_ERR_NOT_PARTITION, "ot_build_tree: leaves do not tile the unit cube");

    int64_t entries = int64_t(1) << (3 * tv.lev[0]), n_sub = 0;
    tv.off[0] = 0;
    for (int t = 1; t < tv.nlev; ++t) {
        tv.off[t] = entries;
        entries += (int64_t)hcnt[t - 1] << (3 * (tv.lev[t] - tv.lev[t - 1]));
        n_sub += (int64_t)hcnt[t - 1];
    }
    if (entries >= (int64_t(1) << 40)) return fail(OT_ERR_CAPACITY, "ot_build_tree: descent table too large");
    // the pool offsets follow the entries, 8-byte aligned, then the root's
    // summary one level up (an eighth of the root: most lookups of points in
    // random order then hit a table small enough for one XCD's L2)
    const int64_t off_at = (entries + 1) & ~int64_t(1);
    // (both pool offsets and block-key bases, int64 each)
    const int64_t sum_at = off_at + 4 * kMaxTabLevels;
    const int64_t sum_cells = tv.lev[0] >= 1 ? (int64_t(1) << (3 * (tv.lev[0] - 1))) : 0;
    // and the anchors of the sub-tables, in the order of their block keys
    const int64_t anc_at = (sum_at + sum_cells + 1) & ~int64_t(1);
    BuildBlock table_block(s);
    if ((rc = table_block.take((size_t)(anc_at + 2 * n_sub) * 4))) return rc;
    uint32_t *table = (uint32_t *)table_block.b.p;
    hipLaunchKernelGGL(k_fill_u32, dim3(2048), dim3(256), 0, s, table, entries, 0xFFFFFFFFu);
    // block keys: the root cubes, then the sub-tables level by level
    int64_t heads[2 * kMaxTabLevels] = {0};
    std::memcpy(heads, tv.off, sizeof(tv.off));
    int64_t *bb = heads + kMaxTabLevels;
    bb[1] = tv.lev[0] >= kBlkBits ? int64_t(1) << (3 * (tv.lev[0] - kBlkBits)) : 0;
    tv.blk1 = (int32_t)bb[1];
    int64_t blocks = bb[1];
    for (int t = 1; t < tv.nlev; ++t) {
        bb[t] = blocks;
        blocks += (int64_t)hcnt[t - 1];
    }
    tv.nblk = (int32_t)blocks;   // at most 8^5 + n_leaves / 8
    OT_HIP(hipMemcpyAsync(table + off_at, heads, sizeof(heads), hipMemcpyHostToDevice, s));
    for (int t = 0; t < tv.nlev; ++t) {
        if (t + 1 < tv.nlev) {
            hipLaunchKernelGGL(k_split_flags, dim3(nblk(n)), dim3(256), 0, s, ks, (const uint8_t *)lvs, n, L,
                               tv.lev[t], flags);
            exclusive_scan(flags, ids, n, stmp, s);
        }
        hipLaunchKernelGGL(k_write_level, dim3(nblk(n)), dim3(256), 0, s, ks, (const uint8_t *)lvs, n, tv,
                           table, t, (const uint32_t *)ids,
                           (uint64_t *)(table + anc_at) + (t + 1 < tv.nlev ? bb[t + 1] - tv.blk1 : 0));
    }
    if (sum_cells)
        hipLaunchKernelGGL(k_root_summary, dim3(nblk(sum_cells)), dim3(256), 0, s, (const uint32_t *)table, sum_cells,
                           tv.lev[0], table + sum_at);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, (uint32_t *)scratch, (int64_t)1, 0u);
    hipLaunchKernelGGL(k_count_value, dim3(1024), dim3(256), 0, s, (const uint32_t *)table, entries, 0xFFFFFFFFu, err);
    OT_HIP(hipGetLastError());
    OT_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, s));
    if (perm_out) OT_HIP(hipMemcpyAsync(perm_out, perm, n * 4, hipMemcpyDeviceToDevice, s));
    OT_HIP(hipStreamSynchronize(s));
    if (herr) return fail(OT_ERR_NOT_PARTITION, "ot_build_tree: descent table has unfilled entries");

    ot_tree *tr = new ot_tree();
    OT_HIP(hipGetDevice(&tr->device));
    tr->cus = 0;
    (void)hipDeviceGetAttribute(&tr->cus, hipDeviceAttributeMultiprocessorCount, tr->device);
    if (tr->cus <= 0) tr->cus = 1;
    tr->l_min = l_min;
    tr->l_max = L;
    tr->periodic = tv.periodic;
    tr->n_leaves = n;
    tr->block_bytes[0] = own.b.bytes;
    tr->block_bytes[1] = table_block.b.bytes;
    (void)own.release();
    (void)table_block.release();
    tr->keys = keys_own;
    tr->levels = lvs;
    tr->table = table;
    tr->table_entries = entries;
    tv.table = tr->table;
    tv.pool_off = (const int64_t *)(tr->table + off_at);
    tv.blk_base = tv.pool_off + kMaxTabLevels;
    tv.blk_anchor = (const uint64_t *)(tr->table + anc_at);
    tv.summary = sum_cells ? tr->table + sum_at : nullptr;
    tv.levels = tr->levels;
    tv.nleaf = (int32_t)n;
    tr->view = tv;
    scratch_trees(tr->device, 1);
    *out = tr;
    return OT_OK;
}

extern "C" int ot_destroy_tree(ot_tree *t)
{
    if (!t) return OT_OK;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(t->device);
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    scratch_trees(t->device, -1);
    if (idle) {
        block_give(Block{t->keys, t->block_bytes[0], t->device});
        block_give(Block{t->table, t->block_bytes[1], t->device});
    } else {
        (void)hipFree(t->keys);
        (void)hipFree(t->table);
    }
    (void)hipSetDevice(cur);
    delete t;
    return OT_OK;
}

extern "C" int ot_tree_info_get(const ot_tree *t, ot_tree_info *info)
{
    if (!t || !info) return fail(OT_ERR_INVALID, "ot_tree_info_get: NULL argument");
    info->n_leaves = t->n_leaves;
    info->l_min = t->l_min;
    info->l_max = t->l_max;
    info->periodic = t->periodic;
    info->table_levels = t->view.nlev;
    info->table_bytes = t->table_entries * 4;
    info->workspace_bytes = spread_ws_bytes(t->n_leaves);
    return OT_OK;
}

extern "C" int ot_tree_leaves(const ot_tree *t, uint64_t *keys_out, uint8_t *levels_out, void *stream)
{
    if (!t) return fail(OT_ERR_INVALID, "ot_tree_leaves: NULL tree");
    hipStream_t s = (hipStream_t)stream;
    if (keys_out) OT_HIP(hipMemcpyAsync(keys_out, t->keys, t->n_leaves * 8, hipMemcpyDeviceToDevice, s));
    if (levels_out) OT_HIP(hipMemcpyAsync(levels_out, t->levels, t->n_leaves, hipMemcpyDeviceToDevice, s));
    return OT_OK;
}
