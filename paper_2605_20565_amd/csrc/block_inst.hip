// One (precision, spreading mode) instantiation of the block pass; the build
// compiles this file once per pair (OT_INST_T, OT_INST_MODE).
#include <algorithm>

#include "batch_plan.h"
#include "block_pass.h"

#ifndef OT_INST_T
#error "OT_INST_T and OT_INST_MODE select the instantiation"
#endif

namespace ot {

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
int enqueue_blocks(const ot_tree *t, BlkWork &w, int ops, const uint64_t *kv, const T *rec, const T *field, T *vel,
                   T *fout, const FxWs &ws, T *grad, hipStream_t s)
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
    return OT_OK;
}

template int enqueue_blocks<OT_INST_T, OT_INST_MODE>(const ot_tree *t, BlkWork &w, int ops, const uint64_t *kv,
                                                    const OT_INST_T *rec, const OT_INST_T *field, OT_INST_T *vel,
                                                    OT_INST_T *fout, const FxWs &ws, OT_INST_T *grad, hipStream_t s);

}  // namespace ot
