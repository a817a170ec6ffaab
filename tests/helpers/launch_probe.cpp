// Runs entry points of liblik without a GPU: the HIP calls they make are
// answered here (this program's definitions come before the runtime's), device
// memory is host memory that no kernel touches, and every kernel launch is
// printed as "name blocks threads stream".
//   batch n_theta n_obs n_particles schedule [kernel cache...]
//   requests n_theta n_obs n_particles schedule [kernel cache...]
//     kernel: LIK_KERNEL_* (generic if not given); the call is made once per
//     kernel cache folder, in this order
//   groups n_groups failing: one engine iteration of n_groups groups beside
//     each other, the launch of group `failing` (-1: none) refused; stream
//     records and waits are printed as "record stream" and "wait stream stream"
//     (an event is named by the stream that recorded it last)
#define __HIP_PLATFORM_AMD__ 1
#include <cxxabi.h>
#include <dlfcn.h>
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "../../include/lik.h"
#include "../../paper_1606_08281_amd/csrc/host.hpp"

namespace {
dim3 g_grid, g_block;
hipStream_t g_stream;
std::map<hipEvent_t, hipStream_t> g_recorded;

std::string kernel_name(const void *fn) {
    Dl_info info;
    if (!dladdr(fn, &info) || !info.dli_sname) return "?";
    int st = 0;
    char *d = abi::__cxa_demangle(info.dli_sname, nullptr, nullptr, &st);
    std::string s = st == 0 ? d : info.dli_sname;
    free(d);
    const size_t at = s.find("k_");
    size_t end = at;
    while (end < s.size() && (isalnum((unsigned char)s[end]) || s[end] == '_')) ++end;
    return at == std::string::npos ? s : s.substr(at, end - at);
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t *s) { *s = (hipStream_t)0x10; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipModuleLoadData(hipModule_t *m, const void *) { *m = (hipModule_t)0x20; return hipSuccess; }
hipError_t hipModuleUnload(hipModule_t) { return hipSuccess; }
hipError_t hipModuleGetFunction(hipFunction_t *f, hipModule_t, const char *name) {
    *f = (hipFunction_t)strdup(name);
    return hipSuccess;
}
hipError_t hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(int *n, hipFunction_t, int, size_t) {
    *n = 24;
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned gx, unsigned, unsigned, unsigned bx,
                                 unsigned, unsigned, unsigned, hipStream_t s, void **, void **) {
    printf("%s %u %u %p\n", (const char *)f, gx, bx, (void *)s);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    g_recorded[e] = s;
    printf("record %p\n", (void *)s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    printf("wait %p %p\n", (void *)s, (void *)g_recorded[e]);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 24;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t s) {
    g_grid = g;
    g_block = b;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, hipStream_t *s) {
    *g = g_grid;
    *b = g_block;
    *n = 0;
    *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **, size_t, hipStream_t s) {
    printf("%s %u %u %p\n", kernel_name(fn).c_str(), g.x, b.x, (void *)s);
    return hipSuccess;
}
}

static int iteration(int n, int failing) {
    lik::EngineArgs e;
    memset(&e, 0, sizeof(e));
    e.f_hi = e.h_max = 1;
    const lik::Net4x8 net{};
    std::vector<lik::GroupLaunch> groups(n);
    for (int g = 0; g < n; ++g) {
        groups[g].umax = g == failing ? 5 : 4;  // no generic kernel has 5 species
        groups[g].rmax = 8;
        groups[g].netargs = &net;
        groups[g].max_items = 1;
    }
    lik::SideStreams side;
    side.fork = (hipEvent_t)0xf0;
    for (int k = 0; k < lik::SideStreams::kN; ++k) {
        side.st[k] = (hipStream_t)(size_t)(0x100 * (k + 1));
        side.join[k] = (hipEvent_t)(size_t)(0xf1 + k);
    }
    const hipError_t err = lik::engine_iteration(e, groups.data(), n, (hipStream_t)0x10, false, &side);
    printf("returned %d\n", (int)err);
    return 0;
}

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "groups" && argc == 4) return iteration(atoi(argv[2]), atoi(argv[3]));
    if (argc < 6 || argc == 7) return 2;
    const int n = atoi(argv[2]), T = atoi(argv[3]), H = atoi(argv[4]), schedule = atoi(argv[5]);
    const int kernel = argc > 6 ? atoi(argv[6]) : LIK_KERNEL_GENERIC;
    const int32_t orders[2] = {0, 1}, stoich[2] = {1, -1};  // immigration and death
    lik_network_t net = nullptr;
    if (lik_create_network(1, 2, orders, stoich, &net) != LIK_OK) return 3;
    lik_tuning tu;
    lik_network_get_tuning(net, &tu);
    tu.schedule = schedule;
    lik_network_set_tuning(net, &tu);
    std::vector<double> theta((size_t)n * 2, 0.0), t(T), y(T, 1.0), ll(n);
    std::vector<int32_t> st(n);
    for (int k = 0; k < T; ++k) t[k] = k + 1.0;
    const int32_t offs[2] = {0, T}, x0[1] = {1};
    const double t0[1] = {0.0};
    const lik_data data = {1, offs, t.data(), y.data(), t0, x0, nullptr};
    lik_obs_model obs;
    memset(&obs, 0, sizeof(obs));
    obs.kind = LIK_OBS_GAUSSIAN;
    obs.n_observed = 1;
    obs.sigma = 1.0;
    int rc = LIK_OK;
    for (int call = argc > 6 ? 7 : 6; rc == LIK_OK && call < (argc > 6 ? argc : 7); ++call) {
        if (argc > 6) setenv("LIK_KERNEL_CACHE", argv[call], 1);
        if (what == "batch") {
            const lik_eval_opts o = {LIK_FP64, kernel, 0, nullptr, 0, 0};
            const size_t bytes = lik_workspace_size(net, n, 1, H);
            void *ws = malloc(bytes);
            rc = lik_eval_batch_device(net, &obs, &o, n, theta.data(), &data, offs, H, 1, ll.data(),
                                       st.data(), nullptr, ws, bytes, nullptr);
        } else {
            lik_request r;
            memset(&r, 0, sizeof(r));
            r.net = net;
            r.obs = obs;
            r.n_theta = n;
            r.theta = theta.data();
            r.data = data;
            r.n_particles = H;
            rc = lik_eval_requests(&r, 1, &tu, kernel, ll.data(), st.data(), nullptr);
        }
    }
    if (rc != LIK_OK) printf("error %d %s\n", rc, lik_last_error());
    return rc == LIK_OK ? 0 : 1;
}
