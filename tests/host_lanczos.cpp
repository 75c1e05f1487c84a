// Eigensolves of a diagonal matrix: what a thread pins it keeps from solve to
// solve and gives back when it ends; without pinned memory a solve is the same.
#include "host_runtime.h"

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <thread>
#include <vector>

#include "../paper_2402_03920_amd/csrc/qsg_transfer.h"

namespace qsg {
int32_t report_error(int32_t code, const char*, ...) { return code; }
hipError_t launch_tm_apply(const TmParams& P, const double* in, double* out, hipStream_t) {
    for (size_t i = 0; i < (size_t)1 << P.n; ++i) out[i] = (double)(i + 1) * in[i];
    return host::launched();
}
hipError_t launch_tm_random(double* v, size_t N, uint64_t, hipStream_t) {
    for (size_t i = 0; i < N; ++i) v[i] = 1.0 + 0.1 * (double)(i % 3);
    return host::launched();
}
hipError_t launch_tm_dots(const double* V, uint32_t nv, size_t N, const double* w, double*,
                          double* h, hipStream_t) {
    for (uint32_t j = 0; j < nv; ++j) {
        h[j] = 0.0;
        for (size_t i = 0; i < N; ++i) h[j] += V[j * N + i] * w[i];
    }
    return host::launched();
}
void update(const double* V, uint32_t nv, size_t N, const double* h, double* w) {
    for (uint32_t j = 0; j < nv; ++j)
        for (size_t i = 0; i < N; ++i) w[i] -= h[j] * V[j * N + i];
}
hipError_t launch_tm_update_dots(const double* V, uint32_t nv, size_t N, const double* h, double* w,
                                 double* p, double* h2, hipStream_t s) {
    update(V, nv, N, h, w);
    return launch_tm_dots(V, nv, N, w, p, h2, s);
}
hipError_t launch_tm_update_norm(const double* V, uint32_t nv, size_t N, const double* h, double* w,
                                 double* p, double* nrm2, hipStream_t s) {
    update(V, nv, N, h, w);
    return launch_tm_dots(w, 1, N, w, p, nrm2, s);
}
hipError_t launch_tm_gather(const double* a, const double* b, const double* c, double* out,
                            hipStream_t) {
    out[0] = *a;
    out[1] = *b;
    out[2] = *c;
    return host::launched();
}
hipError_t launch_tm_scale(const double* w, size_t N, const double* nrm2, double* v, hipStream_t) {
    for (size_t i = 0; i < N; ++i) v[i] = w[i] / std::sqrt(*nrm2);
    return host::launched();
}
hipError_t launch_tm_combine(const double* V, uint32_t nv, size_t N, const double* y, double* out,
                             hipStream_t) {
    for (size_t i = 0; i < N; ++i) {
        out[i] = 0.0;
        for (uint32_t j = 0; j < nv; ++j) out[i] += y[j] * V[j * N + i];
    }
    return host::launched();
}
}  // namespace qsg

bool solves() {
    qsg_tm_desc d{};
    d.L = 2;
    d.parity = 1;
    for (int j = 0; j < 4; ++j) d.jx[j] = d.jy[j] = 1;
    const uint32_t steps = 8;
    const size_t bytes = qsg_tm_lanczos_workspace_bytes(2, steps);
    std::vector<double> ws(bytes / 8 + 1), vec(8);
    double eigs[2], resid[2];
    uint32_t iters = 0;
    return qsg_tm_lanczos(&d, steps, 2, 0.0, 1, ws.data(), bytes, eigs, resid, &iters, vec.data(),
                          nullptr) == QSG_OK &&
           std::fabs(eigs[0] - 8.0) < 1e-12 && std::fabs(eigs[1] - 7.0) < 1e-12 &&
           std::fabs(std::fabs(vec[7]) - 1.0) < 1e-12;
}

int main() {
    bool good = true;
    host::fail_pinned = true;
    std::thread([&] { good = solves(); }).join();
    if (!good) return 1;
    if (host::pinned_frees || host::events) return 2;
    host::fail_pinned = false;
    host::pinned_allocs = 0;
    int frees_between = -1;
    std::thread([&] {
        good = solves() && solves() && solves();
        frees_between = host::pinned_frees;
    }).join();
    std::printf("%d allocations, %d frees between solves, %d at the end, %d events left\n",
                host::pinned_allocs, frees_between, host::pinned_frees, host::events);
    if (!good) return 3;
    if (frees_between != 0) return 4;
    return host::pinned_allocs == 1 && host::pinned_frees == 1 && host::events == 0 ? 0 : 5;
}
