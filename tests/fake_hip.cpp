// A HIP runtime on the host for tests of the library's host side: device memory
// is zeroed host memory, no kernel runs, and every launch is reported to the test
// (with its kernel's name, the current device and its arguments), which returns
// the launch's error.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
typedef int (*LaunchCb)(const char* kernel, int device, void** args);
LaunchCb g_launch = nullptr;
size_t g_limit = ~(size_t)0;   // hipMalloc refuses more than this at once
int g_device = 0;
bool g_capturing = false;
hipError_t g_last = hipSuccess;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_config;
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
hipError_t set(hipError_t e) {
    if (e != hipSuccess) g_last = e;
    return e;
}
hipError_t take(void** p, size_t n) {
    *p = n <= g_limit ? std::calloc(1, n ? n : 1) : nullptr;
    return set(*p ? hipSuccess : hipErrorOutOfMemory);
}
}  // namespace

extern "C" {
char fake_fatbin[64];

void fake_on_launch(LaunchCb cb) { g_launch = cb; }
void fake_malloc_limit(size_t n) { g_limit = n; }
void fake_set_device(int d) { g_device = d; }
void fake_set_capturing(int on) { g_capturing = on != 0; }   // (synchronous calls then fail)
int fake_device() { return g_device; }

void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_config = Config{grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *s = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* host, dim3, dim3, void** args, size_t, hipStream_t) {
    return set(g_launch ? (hipError_t)g_launch(names()[host].c_str(), g_device, args) : hipSuccess);
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetDevice(int* d) {
    *d = g_device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) {
    g_device = d;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof *p);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 6;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char scratch[64];
    *p = scratch;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return g_capturing ? set(hipErrorStreamCaptureUnsupported) : take(p, n); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    if (g_capturing) return set(hipErrorStreamCaptureUnsupported);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t) {
    for (size_t i = 0; i < h; ++i) std::memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)&g_config;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.f;
    return hipSuccess;
}
}  // extern "C"
