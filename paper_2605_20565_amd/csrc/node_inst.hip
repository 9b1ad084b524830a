// One (precision, spreading mode) instantiation of the node-parallel pass; the
// build compiles this file once per pair (OT_INST_T, OT_INST_MODE).
#include <algorithm>

#include "node_pass.h"

#ifndef OT_INST_T
#error "OT_INST_T and OT_INST_MODE select the instantiation"
#endif

namespace ot {

template <typename T, int MODE>
int dispatch_nodes(int ops, const ot_tree *t, hipStream_t s, int64_t n, const void *pos, const void *field,
                   const void *force, int32_t *ids, void *vel, void *fout, void *grad, const FxWs &ws,
                   const int32_t *hid)
{
    constexpr bool f32_sums = std::is_same<T, float>::value && MODE == kModeAtomic;
    const dim3 g((unsigned)((n + kNodePts - 1) / kNodePts)), b(kNodeThreads);
#define OT_NODES(OPSV, PERV)                                                                                       \
    hipLaunchKernelGGL((k_nodes<T, OPSV, MODE, PERV>), g, b, 0, s, t->view, n, (const T *)pos, (const T *)field,    \
                       (const T *)force, ids, (T *)vel, (T *)fout, ws.acc, FxRef{ws.fx, n},        \
                       (T *)grad, hid)
#define OT_CASE(OPSV)                                                                                              \
    case OPSV:                                                                                                     \
        if constexpr (!f32_sums || !((OPSV) & kOpSpread)) {                                                        \
            if (t->view.periodic) OT_NODES(OPSV, true);                                                            \
            else OT_NODES(OPSV, false);                                                                            \
            break;                                                                                                 \
        }                                                                                                          \
        return fail(OT_ERR_INVALID, "sums in FP32 do not take this pass");
    switch (ops) {
        OT_CASE(2) OT_CASE(3) OT_CASE(4) OT_CASE(5) OT_CASE(6) OT_CASE(7)
        OT_CASE(kOpGrad) OT_CASE(kOpGrad | kOpInterp) OT_CASE(kOpGrad | kOpSpread)
    default: return fail(OT_ERR_INVALID, "ops must be a non-empty combination of OT_OP_* bits");
    }
#undef OT_CASE
#undef OT_NODES
    return OT_OK;
}

template <typename T, int MODE>
int enqueue_ranges(const ot_tree *t, int ops, const NodeRanges &nr, unsigned *queue, const uint64_t *kv, const T *rec,
                   const T *field, T *vel, T *fout, const FxWs &ws, T *grad, hipStream_t s)
{
    int64_t most = nr.ranges ? INT32_MAX : (nr.n + nr.pts - 1) / nr.pts;
    const dim3 g((unsigned)std::min<int64_t>(most, 2 * t->cus)), b(kRangeThreads);
#define OT_RANGES(OPSV, M, PERV)                                                                                   \
    hipLaunchKernelGGL((k_node_ranges<T, OPSV, M, PERV>), g, b, 0, s, t->view, nr, queue, kv, rec, field, vel,      \
                       fout, ws.acc, FxRef{ws.fx, nr.n}, grad)
    // passes that do not spread are the same in both modes
#define OT_CASE(OPSV)                                                                                              \
    case OPSV:                                                                                                     \
        if (t->view.periodic) OT_RANGES(OPSV, (((OPSV) & kOpSpread) ? MODE : kModeAtomic), true);                  \
        else OT_RANGES(OPSV, (((OPSV) & kOpSpread) ? MODE : kModeAtomic), false);                                  \
        break;
    switch (ops) {
        OT_CASE(kOpInterp) OT_CASE(kOpSpread) OT_CASE(kOpInterp | kOpSpread)
        OT_CASE(kOpGrad) OT_CASE(kOpGrad | kOpInterp) OT_CASE(kOpGrad | kOpSpread)
    default: return fail(OT_ERR_INVALID, "ops must be a non-empty combination of OT_OP_* bits");
    }
#undef OT_CASE
#undef OT_RANGES
    OT_HIP(hipGetLastError());
    return OT_OK;
}

template int enqueue_ranges<OT_INST_T, OT_INST_MODE>(const ot_tree *t, int ops, const NodeRanges &nr, unsigned *queue,
                                                    const uint64_t *kv, const OT_INST_T *rec, const OT_INST_T *field,
                                                    OT_INST_T *vel, OT_INST_T *fout, const FxWs &ws, OT_INST_T *grad,
                                                    hipStream_t s);

template int dispatch_nodes<OT_INST_T, OT_INST_MODE>(int ops, const ot_tree *t, hipStream_t s, int64_t n,
                                                    const void *pos, const void *field, const void *force,
                                                    int32_t *ids, void *vel, void *fout, void *grad, const FxWs &ws,
                                                    const int32_t *hid);

}  // namespace ot
