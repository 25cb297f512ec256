// A block of the FP32 row pass, row length L (rowc.hip, rowl.hip).
#pragma once
#define C3_ROW_NT C3_ROWC_NT
#include "rowbody.h"

namespace {
template <int L, int MODE>
__device__ __forceinline__ void row_body(const FftArgs &a, const RowTask &task, double *hist) {
    cx<float> *buf = (cx<float> *)c3_rowc_lds;  // 2 L elements
    if (row_idle(a, task)) return;
    // the rows' loads need only the task: they are issued first, and the
    // segment's record and plan load while they are in flight
    cx<float> *ya = (cx<float> *)a.work + task.off_a, *yb = (cx<float> *)a.work + task.off_b;
    row_load<float, L>(buf, ya, yb);
    const SegInfo sg = a.segs[task.seg];
    const FftPlan &p = a.plans[sg.plan];
    const cx<float> *tws = (const cx<float> *)a.twpool + p.twr;
    row_fwd<float, L>(buf, tws);
    row_mid<float, MODE>(a, L, buf, task, sg, p, hist);
    if constexpr (MODE == 0 || MODE == 2) row_inv<float, L>(buf, ya, yb, tws);
}

}  // namespace
