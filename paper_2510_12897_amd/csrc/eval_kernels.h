// Launch entry points of the callback kernels (implemented in the .hip files).
#pragma once

#include <hip/hip_runtime.h>

#include "dev_model.h"

namespace opf {

// Work counts of the two launches of one model (mode 0: callback set,
// 1: J^T v).
SetGrid plan_set(const DevModel& m, const EvalOut& o, int32_t mode);

// One callback set (any subset of f, g, c, J, H) on `stream`: the branch
// phase, then the bus phase.
hipError_t launch_eval_set(const DevModel& m, const EvalOut& o, hipStream_t stream);

// out = J(x)^T v on `stream`; apart: out overlaps neither x nor v.
hipError_t launch_jtprod(const DevModel& m, const double* x, const double* v, double* out, bool apart,
                         hipStream_t stream);

// ---- batched evaluation: one kernel per phase over a list of work items
// (persistent, or one workgroup per item).
struct BatchItem {
    int32_t inst, kind, idx, r;  // instance, task kind, entity chunk / wave / bus, replica
};

struct BatchInst {
    DevModel m;
    int64_t xoff, coff, joff, hoff;  // offsets into the concatenated arrays
};

struct BatchArgs {
    const BatchInst* inst;   // [n_inst] device
    const BatchItem* items;  // [n_items] device
    int32_t n_items;
    const double* X;
    const double* Y;
    const double* sigma;
    double *F, *G, *C, *J, *H;
    int32_t mode;            // 0 = callback set, 1 = J^T v (Y holds V, G holds OUT),
                             // 2 = arc flows into G (X itself, or a copy of a static X)
};

// pd_all, qd_all [n] from rows of row values, stride apart, of pd and qd.
hipError_t launch_load_rows(const double* pd, const double* qd, int64_t n, int64_t row, int64_t stride, double* pd_all,
                            double* qd_all, hipStream_t stream);

// Scratch bytes a model needs per evaluation stream: objective partials,
// then the records (kRecRoom doubles per replica and branch).
size_t scratch_bytes(const DevModel& m);

// Dynamic LDS of a branch phase that writes Jacobian and Hessian, unused: with the 5 KiB
// of staging it leaves six waves on a compute unit (LDS is dealt in 1280-byte
// blocks), which together write no further apart than memory takes well.
// Waves per unit with the items in groups, 48-period set with storage, 200-copy
// N-1 set and 64-scenario batch: 4 29.1, 43.5, 121.3 us; 5 28.5, 43.7, 113.2;
// 6 28.3, 44.4, 113.2; 8 29.2, 46.6, 112.5; 24 29.8, 47.2, 115.7.  The Jacobian
// alone is slower so bounded (batch 44.8 us, 50.7).  The rectangular form's
// items write more and take longer, so that a second round hardly begun costs
// more than the bound gives: 48 periods (2,064 items, 1,536 a round) 34.6 us,
// 32.9 without; from two rounds on it gains too (200 copies, 4,422 items, 60.3
// and 63.1; batch 128.8 and 130.9).
constexpr unsigned kBranchLds = 21 * 1280 - 10 * 64 * 8;
inline unsigned branch_lds(const double* J, const double* H, bool rect, int32_t items) {
    return J && H && (!rect || items >= 2 * 6 * 256) ? kBranchLds : 0;
}

// The batch kernel of phase 0 (branch items) or 1 (bus items) for mode 0
// (callback set), 1 (J^T v) or 2 (flows, phase 0 only, polar only),
// persistent or flat (one workgroup per item), of the polar or the
// rectangular form, with or without storage units and devices in any
// instance (argument: BatchArgs).
void* batch_kernel_fn(int phase, int mode, bool flat, bool rect, bool ext);

// The one-launch batch kernel of callback sets (one workgroup per item:
// branch, generator, storage, device, wide-bus and wave items of every
// instance; bus lanes recompute the branch terms; objective by ticket).
void* batch_single_fn(bool rect, bool ext);

}  // namespace opf
