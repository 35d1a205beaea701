// A stand-in for the HIP runtime, for host-side tests of librbsog without a GPU.
// An executable that includes this file (linked with -Wl,-E against librbsog.so)
// defines the runtime's entry points itself, and the library binds to them:
//   * device and pinned memory is the host's; kernels do nothing, but each launch is
//     shown to `on_launch` (kernel name, grid, the first argument as it was passed);
//   * a copy from the host is only carried out when something waits for it, as the
//     programming model allows: a source that has changed or gone by then is
//     counted in `stale`.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace host_runtime {

struct Launch {
    std::string name;
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
    const void *arg0;
};
struct Copy {
    void *dst;
    const void *src;
    size_t bytes;
    hipStream_t stream;
    std::vector<char> was;
};

// (registered by the library's constructors, before this file's objects)
inline std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> m;
    return m;
}
inline std::vector<Copy> pending;                         // copies from the host nothing has waited for
inline std::function<void(const Launch &)> on_launch;
inline int fail_launch = -1;                              // the launch (counted from 0) that fails, once
inline int launches = 0, stale = 0;
inline std::map<hipStream_t, bool> busy;                  // streams with launches nothing has waited for
inline hipError_t last_error = hipSuccess;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
inline std::vector<Config> configs;

inline bool waited_for_all()
{
    for (const auto &b : busy)
        if (b.second) return false;
    return pending.empty();
}

inline void carry_out(bool all, hipStream_t st)
{
    if (all) busy.clear();
    else busy[st] = false;
    std::vector<Copy> rest;
    for (Copy &c : pending) {
        if (!all && c.stream != st) {
            rest.push_back(c);
            continue;
        }
        if (std::memcmp(c.src, c.was.data(), c.bytes) != 0) {
            ++stale;
            std::printf("a source of %zu bytes changed before its copy was waited for\n", c.bytes);
        }
        std::memcpy(c.dst, c.was.data(), c.bytes);
    }
    pending.swap(rest);
}

}  // namespace host_runtime

extern "C" {
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *)
{
    host_runtime::kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    host_runtime::configs.push_back({grid, block, lds, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    const host_runtime::Config c = host_runtime::configs.back();
    host_runtime::configs.pop_back();
    *grid = c.grid;
    *block = c.block;
    *lds = c.lds;
    *st = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t st)
{
    if (host_runtime::launches++ == host_runtime::fail_launch)
        return host_runtime::last_error = hipErrorLaunchFailure;
    host_runtime::busy[st] = true;
    if (host_runtime::on_launch) host_runtime::on_launch({host_runtime::kernels()[fn], grid, block, lds, st, args[0]});
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = host_runtime::last_error;
    host_runtime::last_error = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "an error"; }
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    if (!*p) return hipErrorOutOfMemory;
    std::memset(*p, 0, n);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorNotSupported; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t st)
{
    if (kind == hipMemcpyHostToDevice) {
        const char *s = (const char *)src;
        host_runtime::pending.push_back({dst, src, n, st, std::vector<char>(s, s + n)});
        return hipSuccess;
    }
    host_runtime::carry_out(false, st);
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind)
{
    host_runtime::carry_out(true, nullptr);
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *dst, int v, size_t n, hipStream_t)
{
    std::memset(dst, v, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    static char streams[64];
    static int n;
    *s = (hipStream_t)(streams + n++);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st)
{
    host_runtime::carry_out(false, st);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    static char event;
    *e = (hipEvent_t)&event;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t)
{
    host_runtime::carry_out(true, nullptr);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.0f;
    return hipSuccess;
}
}
