// The HIP calls of the host runtimes, on a host without a GPU: device memory
// is ordinary memory (reserved, not touched), streams and events are numbers,
// copies run at once.  The drivers of this folder include it before the runtime
// source itself, whose launchers they replace by recorders.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstring>
#include <map>

#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&(x))

static int failures = 0;
static void expect(bool ok, const char* what) {
    if (!ok) {
        std::printf("FAILED: %s\n", what);
        ++failures;
    }
}

namespace stub {
static std::map<void*, size_t> blocks;
static uintptr_t next_id = 1;
static int host_allocs = 0;          // pinned allocations so far
static double clock_us = 0.0;        // what events measure; the drivers advance it
static std::map<hipEvent_t, double> event_us;
template <class T> T id() { return reinterpret_cast<T>(next_id++); }
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) return hipErrorOutOfMemory;
    stub::blocks[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p) {
        munmap(p, stub::blocks.at(p));
        stub::blocks.erase(p);
    }
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    ++stub::host_allocs;
    return hipMalloc(p, n);
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600*, int) { return hipErrorInvalidValue; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = &stub::next_id, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = stub::id<hipStream_t>(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = stub::id<hipGraph_t>(), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = stub::id<hipEvent_t>(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return stub::event_us[e] = stub::clock_us, hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(1e-3 * (stub::event_us[b] - stub::event_us[a]));
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    return *x = stub::id<hipGraphExec_t>(), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}
