// A host stand-in for the HIP runtime and the kernel launchers that the C ABI
// calls: device memory is host memory, a launch runs at once.  Failures are
// forced and calls counted by the program that includes it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>

#include "../include/qsg.h"
#include "../paper_2402_03920_amd/csrc/qsg_internal.h"

namespace host {
int pinned_allocs = 0, pinned_frees = 0, events = 0;
bool fail_pinned = false;
hipError_t last_error = hipSuccess;  // as the runtime: kept until it is asked for
inline hipError_t launched() { return hipGetLastError(); }
}  // namespace host

extern "C" {
hipError_t hipGetLastError() {
    const hipError_t e = host::last_error;
    host::last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "forced"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    ++host::pinned_allocs;
    if (host::fail_pinned) return host::last_error = hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    ++host::pinned_frees;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    ++host::events;
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) {
    --host::events;
    return hipSuccess;
}
}
