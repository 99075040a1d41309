// A HIP runtime of host memory, for checks of the library's host logic without a
// GPU: allocations come from the heap, copies are done at once, kernels are recorded
// and not run.  What a check can ask of it stands in `rt`.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "lb_block.h"

struct Launched {
    std::string kernel;     // mangled name
    bool in_graph;          // recorded by a capture
    lbk::BlockArgs block;   // its arguments, for the block kernels
};

struct HostRuntime {
    std::map<const void*, std::string> names;
    std::vector<Launched> launches;
    int mallocs = 0;              // device allocations so far
    int fail_mallocs = 0;         // that many of the next device allocations fail
    int skip_copies = 0;          // that many copies succeed before
    int fail_copies = 0;          // that many of the next ones fail
    std::vector<unsigned> pinned_flags, event_flags;
    int captures = 0, replays = 0;
    int late_captures = 0;        // begun with work enqueued
    bool pending = false;         // work was enqueued and not waited for
    int destroyed_pending = 0;    // executable graphs destroyed meanwhile
    bool capturing = false;
    hipError_t last_error = hipSuccess;
    int count(const char* part) const {
        int n = 0;
        for (const Launched& l : launches) n += l.kernel.find(part) != std::string::npos;
        return n;
    }
};
inline HostRuntime rt;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    rt.names[f] = name;
}
static struct { dim3 g, b; size_t shm; hipStream_t s; } g_cfg;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t s) {
    g_cfg = {g, b, shm, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, hipStream_t* s) {
    *g = g_cfg.g, *b = g_cfg.b, *shm = g_cfg.shm, *s = g_cfg.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    if (block.x * block.y > 1024 || grid.x * (uint64_t)block.x > 0xffffffffu) {
        rt.last_error = hipErrorInvalidConfiguration;
        return rt.last_error;
    }
    Launched l{rt.names[f], rt.capturing, {}};
    if (l.kernel.find("lb_block") != std::string::npos) l.block = *(const lbk::BlockArgs*)args[0];
    rt.launches.push_back(l);
    rt.pending = rt.pending || !rt.capturing;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = rt.last_error;
    rt.last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "host runtime error"; }
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    *p = nullptr;
    if (rt.fail_mallocs > 0) {
        --rt.fail_mallocs;
        return hipErrorOutOfMemory;
    }
    ++rt.mallocs;
    *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
    rt.pinned_flags.push_back(flags);
    *p = std::calloc(n, 1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    if (rt.skip_copies > 0) {
        --rt.skip_copies;
    } else if (rt.fail_copies > 0) {
        --rt.fail_copies;
        return hipErrorUnknown;
    }
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t) {
    for (size_t y = 0; y < h; ++y) std::memcpy((char*)d + y * dp, (const char*)s + y * sp, w);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free((void*)s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    rt.pending = false;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    if (rt.capturing) return hipErrorIllegalState;
    rt.capturing = true;
    rt.late_captures += rt.pending;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = rt.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    rt.capturing = false;
    ++rt.captures;
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *e = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
    ++rt.replays;
    rt.pending = true;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    rt.destroyed_pending += rt.pending;
    std::free((void*)e);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    std::free((void*)g);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
    rt.event_flags.push_back(flags);
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
    rt.pending = false;
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.f;
    return hipSuccess;
}
}
