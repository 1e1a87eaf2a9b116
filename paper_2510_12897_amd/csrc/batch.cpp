// C-ABI of libopf: batched evaluation of many instances, with a schedule
// autotuner.
//
// An evaluation is two kernel launches on the caller's stream: the branch
// phase of every instance, then the bus phase.  (Launching them from an
// instantiated HIP graph instead cost 4.6 us more per evaluation on the
// 64-scenario mix and on 16 points of the 10k-bus network; the direct
// launches can still be captured into a caller's graph.)  The schedule is
// the grid: with wg_per_cu > 0 each launch is persistent (wg_per_cu
// workgroups per compute unit drain the item list, each XCD's workgroups
// striding through one contiguous range of it); with wg_per_cu = 0 it is
// flat (one workgroup per item, the block index remapped to the same XCD
// ranges).  No schedule
// changes a summation order (segment sums follow the host packing,
// objective partials are per generator chunk and replica and are summed in
// index order), so every schedule produces bitwise the same results as the
// plain per-instance launch.
#include <array>
#include <new>

#include "internal.h"

using namespace opf_internal;

namespace {

// autotuner candidates: the one-launch shape (-1), flat two launches (0),
// then persistent two-launch grids
const int32_t kWgPerCu[] = {-1, 0, 2, 4, 8, 16, 32};

}  // namespace

struct opf_batch_s {
    uint64_t magic = kBatchMagic;
    int device = 0;
    Allocator alloc{};
    int32_t n_inst = 0;
    std::vector<int64_t> xoff, coff, joff, hoff;
    void* arena = nullptr;
    opf::BatchInst* inst = nullptr;  // device
    double* pd_all = nullptr;        // device per-instance loads (NULL if none)
    double* qd_all = nullptr;
    int64_t n_loads = 0;
    opf::BatchItem* items[2][2] = {};  // device item lists, [mode (0 set, 1 J^T v)][phase]
    int32_t n_items[2][2] = {};
    opf::BatchItem* items_single = nullptr;  // the one-launch shape's list (callback sets)
    int32_t n_items_single = 0;
    int32_t wg_per_cu = 0;           // -1: one launch; 0: flat two launches; > 0: persistent two launches
    int32_t n_cu = 256;
    bool rect = false;               // every model is of the rectangular form (else all polar)
    bool ext = false;                // some model has storage units or devices
    bool flat = true;                // every model is static, with branches: x ends with its arcs
};

namespace {

bool valid(const opf_batch_s* b) { return b && b->magic == kBatchMagic; }

// Work items of one phase, one replica each.  Phase 1: the branch chunks,
// then (callback set) the generator chunks, then the storage and device
// chunks of every instance.  Phase 2: big
// buses first (the longest), then the waves of bus segments of every
// instance, then one objective item per instance (callback set) or the
// generator items (J^T v; on a model whose copies share pg, one generator
// per item).  Within a kind, replicas are outermost.
void make_items(const std::vector<opf::DevModel>& dms, int mode, int phase, std::vector<opf::BatchItem>& out) {
    out.clear();
    const int32_t n = (int32_t)dms.size();
    auto each = [&](const opf::DevModel& d, int32_t kind, int32_t count, int32_t j) {
        for (int32_t r = 0; r < d.nrep; r++)
            for (int32_t i = 0; i < count; i++) out.push_back({j, kind, i, r});
    };
    if (phase == 0) {
        for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_BRANCH, dms[j].nbchunks, j);
        if (mode == 0)
            for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_GEN, dms[j].ngchunks, j);
        // storage units and devices (their own rows; J^T v: their entries)
        for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_STOR, dms[j].nschunks, j);
        for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_DEV, dms[j].ndchunks, j);
        return;
    }
    for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_BIG, dms[j].nbig, j);
    for (int32_t j = 0; j < n; j++) each(dms[j], opf::T_WAVE, dms[j].nwaves, j);
    for (int32_t j = 0; j < n; j++) {
        const opf::DevModel& d = dms[j];
        if (mode == 0) {
            out.push_back({j, opf::T_OBJ, 0, 0});
        } else if (d.npg == 1 && d.nrep > 1) {
            for (int32_t k = 0; k < d.G; k++) out.push_back({j, opf::T_GEN, k, 0});
        } else {
            each(d, opf::T_GEN, d.ngchunks, j);
        }
    }
}

int launch(opf_batch_s* b, const opf::BatchArgs& a0, hipStream_t stream) {
    if (a0.mode == 0 && b->wg_per_cu < 0) {
        // one launch: every item of every instance, bus lanes recomputing the
        // branch terms, the objective by each instance's arrival ticket
        opf::BatchArgs a = a0;
        a.inst = b->inst;
        a.items = b->items_single;
        a.n_items = b->n_items_single;
        if (a.n_items == 0) return OPF_OK;
        void* args[1] = {&a};
        const hipError_t e = hipLaunchKernel(opf::batch_single_fn(b->rect, b->ext), dim3(a.n_items),
                                             dim3(opf::kBlock), args, 0, stream);
        return e == hipSuccess ? OPF_OK : hip_err(e, "batch one-launch");
    }
    opf::BatchArgs a[2];
    int32_t grid[2];
    const int lm = a0.mode == 2 ? 0 : a0.mode;  // the flows mode runs the branch items only
    for (int ph = 0; ph < 2; ph++) {
        a[ph] = a0;
        a[ph].inst = b->inst;
        a[ph].items = b->items[lm][ph];
        a[ph].n_items = (a0.mode == 2 && ph == 1) ? 0 : b->n_items[lm][ph];
        // persistent: at least one workgroup per XCD, so every XCD's range is drained
        grid[ph] = b->wg_per_cu <= 0 ? std::max(1, a[ph].n_items)
                                      : std::max(opf::kXcd, std::min(a[ph].n_items, b->n_cu * b->wg_per_cu));
    }
    for (int ph = 0; ph < 2; ph++) {
        if (a[ph].n_items == 0) continue;
        void* args[1] = {&a[ph]};
        const unsigned lds =
            ph == 0 && a0.mode == 0 && b->wg_per_cu <= 0 ? opf::branch_lds(a0.J, a0.H, b->rect, a[ph].n_items) : 0;
        const hipError_t e = hipLaunchKernel(opf::batch_kernel_fn(ph, a0.mode, b->wg_per_cu <= 0, b->rect, b->ext),
                                             dim3(grid[ph]), dim3(opf::kBlock), args, lds, stream);
        if (e != hipSuccess) return hip_err(e, ph == 0 ? "batch branch-phase launch" : "batch bus-phase launch");
    }
    return OPF_OK;
}

}  // namespace

extern "C" {

int opf_batch_create(const opf_model* models, int32_t n_models, const int32_t* inst_model, const double* inst_pd,
                     const double* inst_qd, int32_t n_inst, opf_batch* out) {
    if (!out) return set_err(OPF_E_ARG, "out is NULL");
    *out = nullptr;
    if (!models || n_models < 1 || !inst_model || n_inst < 1)
        return set_err(OPF_E_ARG, "models, inst_model and a positive instance count are required");
    if ((inst_pd == nullptr) != (inst_qd == nullptr))
        return set_err(OPF_E_ARG, "inst_pd and inst_qd must both be given or both be NULL");
    for (int32_t k = 0; k < n_models; k++)
        if (!models[k] || models[k]->magic != kModelMagic)
            return set_err(OPF_E_STATE, "model %d is not a valid handle", k);
    const int dev = models[0]->device;
    for (int32_t k = 1; k < n_models; k++)
        if (models[k]->device != dev) return set_err(OPF_E_ARG, "all models must live on one device");
    for (int32_t k = 1; k < n_models; k++)
        if (models[k]->hm.ly.rect != models[0]->hm.ly.rect)
            return set_err(OPF_E_ARG, "all models of a batch must be of one form (polar or rectangular)");
    for (int32_t j = 0; j < n_inst; j++)
        if (inst_model[j] < 0 || inst_model[j] >= n_models)
            return set_err(OPF_E_ARG, "instance %d names model %d, out of range", j, inst_model[j]);

    opf_batch_s* b = nullptr;
    try {
        b = new opf_batch_s();
        b->device = dev;
        b->rect = models[0]->hm.ly.rect != 0;
        for (int32_t k = 0; k < n_models; k++) {
            const opf::Layout& ly = models[k]->hm.ly;
            if (ly.nrep != 1 || ly.L < 1 || ly.x_q != ly.x_p + 2 * ly.L || ly.n != ly.x_q + 2 * ly.L) b->flat = false;
        }
        for (int32_t k = 0; k < n_models; k++)
            if (models[k]->hm.ly.S > 0 || models[k]->hm.ly.D > 0) b->ext = true;
        b->alloc = current_allocator();
        b->n_inst = n_inst;
        b->xoff.assign(n_inst + 1, 0);
        b->coff.assign(n_inst + 1, 0);
        b->joff.assign(n_inst + 1, 0);
        b->hoff.assign(n_inst + 1, 0);
        for (int32_t j = 0; j < n_inst; j++) {
            const opf::Layout& ly = models[inst_model[j]]->hm.ly;
            b->xoff[j + 1] = b->xoff[j] + ly.n;
            b->coff[j + 1] = b->coff[j] + ly.m();
            b->joff[j + 1] = b->joff[j] + ly.nnzj();
            b->hoff[j + 1] = b->hoff[j] + ly.nnzh;
        }

        // ---- pack: per-instance loads and scratch (zeroed), instance
        // descriptors, item lists
        Packer pk;
        std::vector<int64_t> loff(n_inst + 1, 0);
        std::vector<size_t> o_scr(n_inst, 0);
        std::vector<int32_t> stride(n_inst, 0);
        for (int32_t j = 0; j < n_inst; j++) {
            const opf::HostModel& hm = models[inst_model[j]]->hm;
            loff[j + 1] = loff[j] + (int64_t)hm.ly.N * (hm.ly.T > 1 ? hm.ly.T : 1);
            stride[j] = hm.ly.T > 1 ? hm.ly.N : 0;
            o_scr[j] = pk.reserve(opf::scratch_bytes(models[inst_model[j]]->dm));
        }
        size_t o_pd = 0, o_qd = 0;
        if (inst_pd) {
            o_pd = pk.add(inst_pd, sizeof(double) * loff[n_inst]);
            o_qd = pk.add(inst_qd, sizeof(double) * loff[n_inst]);
        }
        const size_t o_inst = pk.reserve(sizeof(opf::BatchInst) * n_inst);
        std::vector<opf::DevModel> dms(n_inst);
        for (int32_t j = 0; j < n_inst; j++) dms[j] = models[inst_model[j]]->dm;
        size_t lst_off[2][2], lst_single = 0;
        std::vector<opf::BatchItem> items;
        for (int q = 0; q < 4; q++) {  // (mode, phase)
            make_items(dms, q / 2, q % 2, items);
            lst_off[q / 2][q % 2] = pk.add(items);
            b->n_items[q / 2][q % 2] = (int32_t)items.size();
        }
        // the one-launch shape: the callback set's phase-1 items, then its
        // phase-2 items without the objective items (each instance sums its
        // objective by ticket)
        {
            std::vector<opf::BatchItem> all, p2;
            make_items(dms, 0, 0, all);
            make_items(dms, 0, 1, p2);
            for (const opf::BatchItem& w : p2)
                if (w.kind != opf::T_OBJ) all.push_back(w);
            lst_single = pk.add(all);
            b->n_items_single = (int32_t)all.size();
        }

        DeviceGuard dg(dev);
        if (dg.err != hipSuccess) {
            delete b;
            return hip_err(dg.err, "hipSetDevice");
        }
        int ncu = 0;
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && ncu > 0)
            b->n_cu = ncu;
        b->arena = dev_alloc(b->alloc, pk.buf.size());
        if (!b->arena) {
            delete b;
            return set_err(OPF_E_NOMEM, "device allocation of %zu bytes failed", pk.buf.size());
        }
        char* base = static_cast<char*>(b->arena);
        opf::BatchInst* hi = reinterpret_cast<opf::BatchInst*>(pk.at(o_inst));
        for (int32_t j = 0; j < n_inst; j++) {
            opf::BatchInst bi;
            bi.m = dms[j];
            if (inst_pd) {
                bi.m.pd = reinterpret_cast<const double*>(base + o_pd) + loff[j];
                bi.m.qd = reinterpret_cast<const double*>(base + o_qd) + loff[j];
                bi.m.load_stride = stride[j];
            }
            attach_scratch(bi.m, base + o_scr[j]);
            bi.xoff = b->xoff[j];
            bi.coff = b->coff[j];
            bi.joff = b->joff[j];
            bi.hoff = b->hoff[j];
            std::memcpy(&hi[j], &bi, sizeof bi);
        }
        for (int q = 0; q < 4; q++)
            b->items[q / 2][q % 2] = reinterpret_cast<opf::BatchItem*>(base + lst_off[q / 2][q % 2]);
        b->items_single = reinterpret_cast<opf::BatchItem*>(base + lst_single);
        hipError_t e = hipMemcpy(b->arena, pk.buf.data(), pk.buf.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            dev_free(b->alloc, b->arena);
            delete b;
            return hip_err(e, "batch upload");
        }
        if (inst_pd) {
            b->pd_all = reinterpret_cast<double*>(base + o_pd);
            b->qd_all = reinterpret_cast<double*>(base + o_qd);
            b->n_loads = loff[n_inst];
        }
        b->inst = reinterpret_cast<opf::BatchInst*>(base + o_inst);
    } catch (const std::bad_alloc&) {
        delete b;
        return set_err(OPF_E_NOMEM, "host allocation failed");
    }
    *out = b;
    return OPF_OK;
}

int opf_batch_destroy(opf_batch b) {
    if (!b) return OPF_OK;
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    {
        DeviceGuard dg(b->device);
        (void)hipDeviceSynchronize();
        dev_free(b->alloc, b->arena);
    }
    b->magic = 0;
    delete b;
    return OPF_OK;
}

int opf_batch_offsets(opf_batch b, int64_t* xoff, int64_t* coff, int64_t* joff, int64_t* hoff) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    const size_t n = sizeof(int64_t) * (b->n_inst + 1);
    if (xoff) std::memcpy(xoff, b->xoff.data(), n);
    if (coff) std::memcpy(coff, b->coff.data(), n);
    if (joff) std::memcpy(joff, b->joff.data(), n);
    if (hoff) std::memcpy(hoff, b->hoff.data(), n);
    return OPF_OK;
}

int opf_batch_schedule(opf_batch b, int32_t* wg_per_cu) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (wg_per_cu) *wg_per_cu = b->wg_per_cu;
    return OPF_OK;
}

int opf_batch_set_schedule(opf_batch b, int32_t wg_per_cu) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (wg_per_cu < -1 || wg_per_cu > 64) return set_err(OPF_E_ARG, "wg_per_cu must be in [-1, 64]");
    b->wg_per_cu = wg_per_cu;
    return OPF_OK;
}

int opf_batch_eval(opf_batch b, const double* X, const double* Y, const double* sigma, double* F, double* G,
                   double* C, double* J, double* H, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!X) return set_err(OPF_E_ARG, "X must be non-NULL");
    if (H && (!Y || !sigma)) return set_err(OPF_E_ARG, "Y and sigma must be non-NULL when H is requested");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    opf::BatchArgs a{};
    a.X = X; a.Y = Y; a.sigma = sigma; a.F = F; a.G = G; a.C = C; a.J = J; a.H = H;
    a.mode = 0;
    return launch(b, a, static_cast<hipStream_t>(stream));
}

int opf_batch_jtprod(opf_batch b, const double* X, const double* V, double* OUT, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!X || !V || !OUT) return set_err(OPF_E_ARG, "X, V and OUT must be non-NULL");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    opf::BatchArgs a{};
    a.X = X; a.Y = V; a.G = OUT;
    a.mode = 1;
    return launch(b, a, static_cast<hipStream_t>(stream));
}

int opf_batch_set_loads(opf_batch b, const double* pd, const double* qd, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!b->pd_all) return set_err(OPF_E_STATE, "the batch was created without per-instance loads");
    if (!pd || !qd) return set_err(OPF_E_ARG, "pd and qd must be non-NULL");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t bytes = sizeof(double) * (size_t)b->n_loads;
    hipError_t e = hipMemcpyAsync(b->pd_all, pd, bytes, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b->qd_all, qd, bytes, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return hip_err(e, "load copy");
    return OPF_OK;
}

int opf_batch_set_load_rows(opf_batch b, const double* pd, const double* qd, int64_t row, int64_t stride,
                            void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!b->pd_all) return set_err(OPF_E_STATE, "the batch was created without per-instance loads");
    if (!pd || !qd) return set_err(OPF_E_ARG, "pd and qd must be non-NULL");
    if (row < 1 || stride < 0 || b->n_loads % row) return set_err(OPF_E_ARG, "rows of %lld values do not make up the loads", (long long)row);
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    const hipError_t e = opf::launch_load_rows(pd, qd, b->n_loads, row, stride, b->pd_all, b->qd_all,
                                               static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_err(e, "load rows launch");
    return OPF_OK;
}

int opf_batch_flows_to(opf_batch b, const double* X, double* OUT, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!X || !OUT) return set_err(OPF_E_ARG, "X and OUT must be non-NULL");
    if (b->rect || !b->flat) return set_err(OPF_E_ARG, "opf_batch_flows_to takes static polar models only");
    // one instance's copy would race with another's reads
    const uintptr_t xa = reinterpret_cast<uintptr_t>(X), oa = reinterpret_cast<uintptr_t>(OUT);
    const size_t bytes = sizeof(double) * (size_t)b->xoff.back();
    if (xa != oa && xa < oa + bytes && oa < xa + bytes)
        return set_err(OPF_E_ARG, "OUT must be X itself or apart from it");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    opf::BatchArgs a{};
    a.X = X;
    a.G = OUT;
    a.mode = 2;
    return launch(b, a, static_cast<hipStream_t>(stream));
}

int opf_batch_flows(opf_batch b, double* X, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    if (!X) return set_err(OPF_E_ARG, "X must be non-NULL");
    if (b->rect) return set_err(OPF_E_ARG, "opf_batch_flows takes polar models only");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    opf::BatchArgs a{};
    a.X = X;
    a.G = X;
    a.mode = 2;
    return launch(b, a, static_cast<hipStream_t>(stream));
}

int opf_batch_tune(opf_batch b, void* stream) {
    if (!valid(b)) return set_err(OPF_E_STATE, "invalid or destroyed batch handle");
    DeviceGuard dg(b->device);
    if (dg.err != hipSuccess) return hip_err(dg.err, "hipSetDevice");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t n = b->xoff.back(), m = b->coff.back(), nj = b->joff.back(), nh = b->hoff.back();
    const size_t bytes = sizeof(double) * (size_t)(2 * n + 2 * m + nj + nh + 2 * b->n_inst);
    void* buf = dev_alloc(b->alloc, bytes);
    if (!buf) return set_err(OPF_E_NOMEM, "tuning buffers (%zu bytes)", bytes);
    double* p = static_cast<double*>(buf);
    double *X = p, *G = X + n, *Y = G + n, *C = Y + m, *J = C + m, *H = J + nj, *sg = H + nh, *F = sg + b->n_inst;
    int rc = OPF_OK;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const int32_t keep_wg = b->wg_per_cu;
    constexpr int kCand = (int)(sizeof(kWgPerCu) / sizeof(kWgPerCu[0]));
    // each candidate's best of three rounds, the rounds interleaved over the
    // candidates: a transient slowdown (another process, a profiler starting)
    // then cannot decide the choice
    std::array<float, kCand> best_ms;
    best_ms.fill(1e30f);
    do {
        hipError_t e = hipMemsetAsync(buf, 0, bytes, s);
        if (e == hipSuccess) e = hipEventCreate(&e0);
        if (e == hipSuccess) e = hipEventCreate(&e1);
        if (e != hipSuccess) {
            rc = hip_err(e, "tuning setup");
            break;
        }
        for (int round = 0; round < 3 * kCand && rc == OPF_OK; round++) {
            const int ci = round % kCand;
            const int32_t wg = kWgPerCu[ci];
            b->wg_per_cu = wg;
            opf::BatchArgs a{};
            a.X = X; a.Y = Y; a.sigma = sg; a.F = F; a.G = G; a.C = C; a.J = J; a.H = H;
            for (int w = 0; w < 2 && rc == OPF_OK; w++) rc = launch(b, a, s);
            if (rc) break;
            (void)hipEventRecord(e0, s);
            const int reps = 5;
            for (int w = 0; w < reps && rc == OPF_OK; w++) rc = launch(b, a, s);
            if (rc) break;
            (void)hipEventRecord(e1, s);
            e = hipEventSynchronize(e1);
            if (e != hipSuccess) {
                rc = hip_err(e, "tuning run");
                break;
            }
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            best_ms[ci] = std::min(best_ms[ci], ms);
        }
    } while (false);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(s);
    dev_free(b->alloc, buf);
    if (rc) {
        b->wg_per_cu = keep_wg;
        return rc;
    }
    int ci_best = 0;
    for (int ci = 1; ci < kCand; ci++)
        if (best_ms[ci] < best_ms[ci_best]) ci_best = ci;
    b->wg_per_cu = kWgPerCu[ci_best];
    return OPF_OK;
}

}  // extern "C"
