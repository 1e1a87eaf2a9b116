// Host driver for prox_train_step's order of launches (CPU only): the entry
// point's own code over stand-ins for the kernel launchers, which count
// themselves, keep the step count as the kernels do, and fail from a chosen
// one on.  Built and run by tests/test_train_step_failures.py.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "internal.h"
#include "proxy_kernels.h"

namespace {
int g_launch = 0, g_fail_at = 0;
hipError_t launch() { return ++g_launch >= g_fail_at && g_fail_at ? hipErrorLaunchFailure : hipSuccess; }
}  // namespace

namespace opf_internal {
int set_err(int code, const char*, ...) { return code; }
int hip_err(hipError_t, const char*) { return OPF_E_HIP; }
}  // namespace opf_internal

namespace opf {
int prox_gemm_splits(int, int, int) { return 2; }
bool prox_loss_fused_size(int, int, int) { return true; }
hipError_t prox_gemm_mixed(int, const void*, bool, int, const void*, bool, int, float*, int, int, int, int,
                           const float*, void*, bool, int, int, float*, hipStream_t) { return launch(); }
hipError_t prox_gemm_split_parts(int, const void*, bool, int, const void*, bool, int, int, int, int, int, float*,
                                 hipStream_t) { return launch(); }
hipError_t prox_gemm_gelu_bwd(const void*, bool, int, const void*, bool, int, const float*, int, void*, int, int, int,
                              int, float*, hipStream_t) { return launch(); }
hipError_t prox_gelu_bwd(const float*, const float*, float*, int64_t, hipStream_t) { return launch(); }
hipError_t prox_to_bf16(const float*, int64_t, void*, hipStream_t) { return launch(); }
hipError_t prox_loss_fused(const DevModel&, const ProxBox&, const ProxRows&, const ProxPerm&, const float*,
                           const double*, int, double, double, double*, double*, double*, double*, double*,
                           hipStream_t, float*, double) { return launch(); }
hipError_t prox_colsum_first(const float*, int, int, float*, void*, const int32_t* step, int32_t* next, hipStream_t) {
    const hipError_t e = launch();
    if (e == hipSuccess && next) *next = *step + 1;
    return e;
}
hipError_t prox_update(UpdateLayers, float*, float*, float*, void*, float, float, float, float, const int32_t* count,
                       int32_t* step, hipStream_t) {
    const hipError_t e = launch();
    if (e == hipSuccess && step) *step = *count;
    return e;
}
// entry points of the same file that the driver does not call
hipError_t prox_colsum(const float*, int, int, float*, float*, float, hipStream_t) { std::abort(); }
hipError_t prox_colsum_parts(const float*, int, int, float*, float, hipStream_t) { std::abort(); }
hipError_t prox_adam(float*, const float*, float*, float*, int64_t, float, float, float, float, int, void*,
                     hipStream_t) { std::abort(); }
hipError_t prox_adam_dev(float*, const float*, float*, float*, int64_t, float, float, float, float, int32_t*, void*,
                         hipStream_t) { std::abort(); }
hipError_t prox_squash_fwd(const float*, int, const ProxBox&, double*, int64_t, bool, hipStream_t) { std::abort(); }
hipError_t prox_squash_bwd(const float*, int, const ProxBox&, const double*, const double*, const double*, double,
                           int64_t, float*, float, hipStream_t) { std::abort(); }
hipError_t prox_penalty(const double*, const double*, const double*, double, const ProxRows&, double, int, double*,
                        double*, double*, double*, int, hipStream_t) { std::abort(); }
hipError_t prox_vjp_weights(const double*, const double*, const double*, const ProxRows&, int, double*, hipStream_t) {
    std::abort();
}
hipError_t prox_vjp_sum(const double*, const double*, const double*, const ProxObj&, double, const double*, int,
                        int64_t, int64_t, double*, hipStream_t) { std::abort(); }
hipError_t prox_loss_bwd(const float*, int, const ProxBox&, const ProxObj&, const double*, const double*, double,
                         const double*, int64_t, float*, hipStream_t) { std::abort(); }
hipError_t prox_scale_rows(const double*, const double*, double, int, int, float*, hipStream_t) { std::abort(); }
hipError_t prox_sample_loads(const double*, const double*, const double*, double, int, int, double*, float*,
                             hipStream_t) { std::abort(); }
}  // namespace opf

int main() {
    opf_model_s model;
    opf::Layout& ly = model.hm.ly;
    ly.N = 4;
    ly.G = 2;
    ly.L = 4;
    ly.nrep = 1;
    ly.x_va = 0;
    ly.x_vm = 4;
    ly.x_pg = 8;
    ly.x_qg = 10;
    ly.x_p = 12;
    ly.x_q = 20;
    ly.n = 28;
    const double2 br{};
    model.fuse_br = &br;
    int bad = 0;
    // one update launch, and two (more layers than one takes); a hidden width of 8 and of 12 values
    for (int depth : {1, 8})
        for (int width : {8, 12}) {
            std::vector<int32_t> dims{8};
            for (int k = 0; k < depth; k++) dims.push_back(width);
            dims.push_back(12);
            alignas(16) static float par[8192], m1[8192], m2[8192], feats[64];
            int32_t step = 41;
            prox_mlp_desc d{(int32_t)dims.size() - 1, dims.data(), par, nullptr, m1, m2, &step};
            int64_t bytes = 0;
            if (prox_train_step_bytes(&d, 8, &bytes) != OPF_OK) return 2;
            std::vector<char> raw((size_t)bytes + 256);
            char* work = raw.data() + (256 - reinterpret_cast<uintptr_t>(raw.data()) % 256) % 256;
            double loads[64] = {}, loss[8], cvio[8];
            auto run = [&](int fail_at) {
                g_launch = 0;
                g_fail_at = fail_at;
                return prox_train_step(&model, &d, feats, loads, 8, 0.3, 1.0, 1.0, 1e-3f, 0.9f, 0.999f, 1e-8f, work,
                                       bytes, loss, cvio, nullptr, nullptr);
            };
            if (run(0) != OPF_OK || step != 42) {
                std::printf("a whole step: count %d\n", step);
                return 3;
            }
            const int launches = g_launch;
            for (int f = 1; f <= launches; f++) {
                if (run(f) != OPF_E_HIP || step != 42) {
                    std::printf("depth %d width %d: launch %d of %d failing leaves the count at %d\n", depth, width, f,
                                launches, step);
                    bad++;
                    step = 42;
                }
            }
        }
    if (bad) return 1;
    std::printf("train step driver: ok\n");
    return 0;
}
