// A stand-in for the HIP runtime calls that libccl.so makes, for CPU tests of
// its host side: memory is handed out as addresses that nothing is behind (no
// kernel runs), and every allocation, free, wait and launch is logged.  Loaded
// with global symbols before the library, so that its calls resolve here.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <unistd.h>

#include "ccl_kernels.h"

static std::mutex g_mu;
static std::string g_log;
static std::map<const void*, std::string> g_names;  // kernel stub -> mangled name
static uintptr_t g_next = uintptr_t(1) << 44;
static std::atomic<int64_t> g_limit{INT64_MAX};  // larger allocations fail
static std::atomic<int> g_delay_us{0};           // every launch takes this long
static std::atomic<int> g_threads{0};

static int thread_no()
{
    static thread_local const int n = g_threads++;
    return n;
}
static void note(const char* what, hipStream_t st, const void* p, int64_t v = 0)
{
    char line[512];
    snprintf(line, sizeof line, "%s %d %llx %llx %lld\n", what, thread_no(),
             (unsigned long long)(uintptr_t)st, (unsigned long long)(uintptr_t)p, (long long)v);
    std::lock_guard<std::mutex> lk(g_mu);
    g_log += line;
}

extern "C" {

void rec_limit(int64_t bytes) { g_limit = bytes; }
void rec_delay_us(int us) { g_delay_us = us; }
// Log so far ("what thread stream pointer value", one event a line), which is then cleared.
int64_t rec_take(char* out, int64_t cap)
{
    std::lock_guard<std::mutex> lk(g_mu);
    const int64_t n = (int64_t)g_log.size();
    if (n < cap) {
        std::memcpy(out, g_log.c_str(), (size_t)n + 1);
        g_log.clear();
    }
    return n;
}

void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*)
{
    g_names[host] = name;
}

static thread_local struct {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} g_call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t st)
{
    g_call = {grid, block, shared, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* st)
{
    *grid = g_call.grid;
    *block = g_call.block;
    *shared = g_call.shared;
    *st = g_call.stream;
    return hipSuccess;
}
// Kernels over a workspace: pointer = the workspace; those over images: value =
// the merge groups.
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t st)
{
    if (g_delay_us) usleep((useconds_t)g_delay_us);
    const std::string& name = g_names[f];
    const char* k = strstr(name.c_str(), "k_");
    size_t n = 0;
    while (k && k[n] && (k[n] == '_' || (k[n] >= 'a' && k[n] <= 'z'))) ++n;
    const std::string what = "launch:" + std::string(k ? k : "?", k ? n : 1);
    if (name.find("VolWs") != std::string::npos) {
        note(what.c_str(), st, static_cast<const ccl::VolWs*>(args[1])->bits);
    } else if (name.find("BatchArgs") != std::string::npos &&
               name.find("Workspace") != std::string::npos) {
        note(what.c_str(), st, static_cast<const ccl::Workspace*>(args[1])->bits,
             static_cast<const ccl::BatchArgs*>(args[0])->ngroups);
    } else {
        note(what.c_str(), st, nullptr);
    }
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t bytes)
{
    *p = nullptr;
    if ((int64_t)bytes > g_limit) {
        note("refused", nullptr, nullptr, (int64_t)bytes);
        return hipErrorOutOfMemory;
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        *p = reinterpret_cast<void*>(g_next);
        g_next += (bytes + 0xffff) & ~size_t(0xffff);
    }
    note("malloc", nullptr, *p, (int64_t)bytes);
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    note("free", nullptr, p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned)
{
    *p = malloc(bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st)
{
    note("wait", st, nullptr);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    note("wait_device", nullptr, nullptr);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void*, size_t bytes, hipMemcpyKind, hipStream_t st)
{
    note("copy", st, dst, (int64_t)bytes);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 4;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = reinterpret_cast<void*>(uintptr_t(1) << 40);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = reinterpret_cast<hipEvent_t>(uintptr_t(1));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.f;
    return hipSuccess;
}

}  // extern "C"
