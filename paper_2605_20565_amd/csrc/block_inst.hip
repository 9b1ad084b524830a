// One (precision, spreading mode) instantiation of the block pass; the build
// compiles this file once per pair (OT_INST_T, OT_INST_MODE).
#include <algorithm>

#include "batch_plan.h"
#include "block_pass.h"

#ifndef OT_INST_T
#error "OT_INST_T and OT_INST_MODE select the instantiation"
#endif

namespace ot {

// Gradients of points whose vector is not finite, over the block pass's, on
// trees with walls: a node beyond a wall has field 0 in a block's grid, which
// an infinite vector turns into NaN, and the per-point pass drops the node.
// st: the run's fixed-point state, which knows whether there is such a vector
// (null: every vector is read here, 12 bytes a point).  In the block pass the
// same sums cost 100 -> 168 registers and spills (2 M points, FP64, both outputs
// 505 -> 704 us), and a flag set there still 231 -> 288 us of an FP32 gradient.
template <typename T>
static __global__ __launch_bounds__(256) void k_grad_again(TreeView tv, const FxState *__restrict__ st, int64_t n,
                                                           const T *__restrict__ pos, const T *__restrict__ vec,
                                                           const T *__restrict__ field, T *__restrict__ grad)
{
    if (st && st->nonfinite == 0ull) return;
    DirectSink<T, kModeAtomic> sink{nullptr, nullptr, 0.0};
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const T F[3] = {vec[3 * k], vec[3 * k + 1], vec[3 * k + 2]};
        if (isfinite(F[0]) && isfinite(F[1]) && isfinite(F[2])) continue;
        const T X[3] = {pos[3 * k], pos[3 * k + 1], pos[3 * k + 2]};
        track_point_at<T, kOpGrad, false>(tv, k, false, 0ull, X, 3, field, vec, (int32_t *)nullptr, (T *)nullptr, sink,
                                          grad, (const int32_t *)nullptr, F);
    }
}

template <typename T, int MODE>
static const void *block_fn(int ops, bool root)
{
    // passes that do not spread are the same in both modes
#define OT_FN(OPSV)                                                                                                 \
    case OPSV: {                                                                                                    \
        constexpr int M = ((OPSV) & kOpSpread) ? MODE : kModeAtomic;                                                \
        return root ? (const void *)k_block<T, M, OPSV, true> : (const void *)k_block<T, M, OPSV, false>;           \
    }
    switch (ops) {
        OT_FN(kOpInterp)
        OT_FN(kOpSpread)
        OT_FN(kOpInterp | kOpSpread)
        OT_FN(kOpGrad)
        OT_FN(kOpGrad | kOpInterp)
        OT_FN(kOpGrad | kOpSpread)
    default: return nullptr;
    }
#undef OT_FN
}

template <typename T, int MODE>
int enqueue_blocks(const ot_tree *t, BlkWork &w, int ops, const uint64_t *kv, const T *rec, const T *pos, const T *vec,
                   const T *field, T *vel, T *fout, const FxWs &ws, T *grad, hipStream_t s)
{
    const TreeView &tv = t->view;
    enqueue_bounds(t, w, kv, s);
    for (int root = 1; root >= 0; --root) {
        const BlkTile *tiles = root ? w.root_tiles : w.sub_tiles;
        const unsigned *count = w.words + (root ? kBlkRootTiles : kBlkSubTiles);
        unsigned *queue = w.words + (root ? kBlkRootQueue : kBlkSubQueue);
        if (root ? tv.blk1 == 0 : tv.nblk == tv.blk1) continue;
        TreeView tvv = tv;
        unsigned long long *acc = ws.acc;
        FxRef fx{ws.fx, w.n};
        bool stream = 3 * w.n * (int64_t)sizeof(T) > kBlkStreamBytes;
        void *args[] = {&tvv, &tiles, &count, &queue, &kv, &rec, &field, &vel, &fout, &acc, &fx, &grad, &stream};
        OT_HIP(hipLaunchKernel(block_fn<T, MODE>(ops, root), dim3(w.grid),
                               dim3(root ? BlkThreads<T, true>::value : BlkThreads<T, false>::value), args, 0, s));
    }
    if ((ops & kOpGrad) && !tv.periodic) {
        const FxState *st = MODE == kModeFixed && (ops & kOpSpread) ? ws.fx : nullptr;
        hipLaunchKernelGGL(k_grad_again<T>, dim3((unsigned)std::min<int64_t>((w.n + 255) / 256, st ? 512 : 4096)), dim3(256),
                           0, s, tv, st, w.n, pos, vec, field, grad);
    }
    return OT_OK;
}

template int enqueue_blocks<OT_INST_T, OT_INST_MODE>(const ot_tree *t, BlkWork &w, int ops, const uint64_t *kv,
                                                    const OT_INST_T *rec, const OT_INST_T *pos, const OT_INST_T *vec,
                                                    const OT_INST_T *field, OT_INST_T *vel, OT_INST_T *fout,
                                                    const FxWs &ws, OT_INST_T *grad, hipStream_t s);

}  // namespace ot
