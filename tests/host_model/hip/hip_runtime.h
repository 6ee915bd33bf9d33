// What the library's sources need of the HIP runtime and language, on the CPU, for
// the tests (tests/test_host_kernels.py): the same kernels, launchers and host code
// run with no GPU, on memory that shows every access out of range.
//
// * hipMalloc: whole pages between two inaccessible ones, the allocation at the end
//   (or, host_side(0), at the start) of them, so the first byte past it (before it)
//   faults; filled with NaN; the slack beside it is checked for stores.
// * LDS (__shared__, rewritten to host::lds): the same, NaN at each block's start.
// * A block's threads are fibres that run from one barrier to the next in turn, in
//   ascending or (host_order(1)) descending order: results that differ between the
//   two need a barrier that is not there.
// * Launches run at once; while a stream is captured they are kept and run by
//   hipGraphLaunch.  Streams and events order nothing (everything is in order).
// * __umul24 checks that its operands and its product fit.
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __constant__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct alignas(8) float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(16) double2 { double x, y; };
struct alignas(8) uint2 { unsigned x, y; };
struct alignas(16) uint4 { unsigned x, y, z, w; };
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline double2 make_double2(double x, double y) { return {x, y}; }
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};

// ---- runtime ----------------------------------------------------------------
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorInvalidConfiguration = 9 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
constexpr unsigned hipEventDisableTiming = 2, hipEventDisableSystemFence = 4, hipStreamNonBlocking = 1,
                   hipHostMallocMapped = 2;
struct HostGraph {
    std::vector<std::function<void()>> nodes;
};
using hipStream_t = struct HostStream*;
using hipEvent_t = struct HostEvent*;
using hipGraph_t = HostGraph*;
using hipGraphExec_t = HostGraph*;

namespace host {
void* guarded(size_t bytes);
void release(void* p);
void* block_lds(void*& cell, size_t bytes);
void launch(const char* name, dim3 grid, dim3 block, const std::function<void()>& thread);
void barrier();
double wave_xor(double v, int mask);
bool wave_any(bool v);
[[noreturn]] void stop(const char* what);
extern HostGraph* capture;

struct Index {
    unsigned x, y, z;
};
extern Index thread, block, block_dim, grid_dim;

template <typename V, typename Site>
V& lds(Site) {
    static void* cell = nullptr;
    return *(V*)block_lds(cell, sizeof(V));
}

// k<<<grid, block, 0, stream>>>(args) as launcher("k", &k, grid, block, 0, stream)(args)
template <typename... P>
struct Launcher {
    const char* name;
    void (*k)(P...);
    dim3 g, b;
    void operator()(P... a) const {
        auto f = k;
        launch(name, g, b, [=] { f(a...); });
    }
};
template <typename... P>
Launcher<P...> launcher(const char* name, void (*k)(P...), dim3 g, dim3 b, int, hipStream_t) {
    return {name, k, g, b};
}
}  // namespace host

#define threadIdx host::thread
#define blockIdx host::block
#define blockDim host::block_dim
#define gridDim host::grid_dim

inline void __syncthreads() { host::barrier(); }
inline double __shfl_xor(double v, int mask, int) { return host::wave_xor(v, mask); }
inline int __any(int v) { return host::wave_any(v != 0); }
inline unsigned __umul24(unsigned a, unsigned b) {
    if (a >> 24 || b >> 24 || ((unsigned long)a * b) >> 32) host::stop("__umul24 of values that do not fit");
    return a * b;
}
inline double rsqrt(double v) { return 1.0 / std::sqrt(v); }
using std::fmax;
using std::fmin;

inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "error of the CPU runtime"; }
template <typename V>
inline hipError_t hipMalloc(V** p, size_t n) {
    *p = (V*)host::guarded(n);
    return hipSuccess;
}
inline hipError_t hipFree(void* p) {
    host::release(p);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
inline hipError_t hipHostFree(void* p) { return hipFree(p); }
inline hipError_t hipHostGetDevicePointer(void** d, void* p, unsigned) {
    *d = p;
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    if (host::capture)
        host::capture->nodes.push_back([=] { std::memmove(d, s, n); });
    else
        std::memmove(d, s, n);
    return hipSuccess;
}
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    return hipMemcpyAsync(d, s, n, k, nullptr);
}
inline hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    if (host::capture) host::stop("hipMemsetAsync under capture");
    std::memset(d, v, n);
    return hipSuccess;
}
inline hipError_t hipMemset(void* d, int v, size_t n) { return hipMemsetAsync(d, v, n, nullptr); }
#define HIP_SYMBOL(s) ((void*)&(s))
inline hipError_t hipGetSymbolAddress(void** p, void* s) {
    *p = s;
    return hipSuccess;
}
inline hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
    std::free((void*)s);
    return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
inline hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
inline hipError_t hipEventDestroy(hipEvent_t e) {
    std::free((void*)e);
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = host::capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    if (host::capture) return hipErrorInvalidValue;
    host::capture = new HostGraph();
    return hipSuccess;
}
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = host::capture;
    host::capture = nullptr;
    return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, void*, char*, size_t) {
    *e = new HostGraph(*g);
    return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) {
    delete g;
    return hipSuccess;
}
inline hipError_t hipGraphExecDestroy(hipGraphExec_t g) { return hipGraphDestroy(g); }
inline hipError_t hipGraphLaunch(hipGraphExec_t g, hipStream_t) {
    for (auto& n : g->nodes) n();
    return hipSuccess;
}
inline hipError_t hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
    const void* table = *(const void**)args[0];  // the job-table kernels' one argument
    auto k = (void (*)(const void*))fn;
    host::launch("job-table kernel", g, b, [=] { k(table); });
    return hipSuccess;
}
