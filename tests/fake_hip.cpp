// A stand-in for the HIP runtime that runs nothing: it carries the runtime's soname, so the library
// under test binds to it when it is loaded first, and lists every kernel launch (name, grid, block, first
// arguments). Memory calls succeed without touching device addresses. Tests of the host code use it on
// machines without a GPU: which launches a call makes, and what a call does when one of them fails.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

std::map<const void *, std::string> g_names;
struct Launch {
    std::string name;
    uint64_t grid, block, arg[8];
};
std::vector<Launch> g_log;
std::string g_fail;      // launches of kernels whose name contains this fail
int g_fail_after = 0;    // ... after this many good ones
bool g_capturing = false;
std::vector<double> g_result;                // what the next sums over work-groups give
std::vector<std::pair<char *, size_t>> g_host;  // pinned host memory
hipError_t g_last = hipSuccess;
thread_local struct {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} g_config;

// Arguments of 8 bytes or less that may be read, by kernel; at least the first two of every kernel.
int readable(const std::string &name)
{
    if (name.find("k_tile") != std::string::npos) return 8;
    if (name.find("k_batch_tile") != std::string::npos) return 7;
    if (name.find("k_sum_partials") != std::string::npos) return 4;
    if (name.find("k_reduce_partials") != std::string::npos) return 3;
    return 2;
}

// Bytes of argument i that a kernel takes as a 32-bit number.
bool is_int(const std::string &name, int i)
{
    if (name.find("k_tile") != std::string::npos) return i == 7;
    if (name.find("k_batch_tile") != std::string::npos) return i >= 5;
    if (name.find("k_sum_partials") != std::string::npos) return i == 1 || i == 2;
    if (name.find("k_reduce_partials") != std::string::npos) return i == 1;
    return false;
}

hipError_t set(hipError_t e)
{
    if (e != hipSuccess) g_last = e;
    return e;
}

}  // namespace

extern "C" {

// ---- controls for the tests ----
void fake_clear() { g_log.clear(); }
void fake_capture(int on) { g_capturing = on != 0; }
void fake_fail(const char *name, int after)
{
    g_fail = name ? name : "";
    g_fail_after = after;
}
void fake_result(const double *v, int n) { g_result.assign(v, v + n); }
int fake_count() { return (int)g_log.size(); }
const char *fake_name(int i) { return g_log[(size_t)i].name.c_str(); }
uint64_t fake_grid(int i) { return g_log[(size_t)i].grid; }
uint64_t fake_block(int i) { return g_log[(size_t)i].block; }
uint64_t fake_arg(int i, int a) { return g_log[(size_t)i].arg[a]; }

// ---- the runtime ----
static void *g_module;
void **__hipRegisterFatBinary(const void *) { return &g_module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *,
                           int *)
{
    int st = 0;
    char *d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    g_names[host] = d ? d : device;
    std::free(d);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_config = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = g_config.grid;
    *block = g_config.block;
    *shared = g_config.shared;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t)
{
    Launch l;
    l.name = g_names[f];
    l.grid = (uint64_t)grid.x * grid.y * grid.z;
    l.block = (uint64_t)block.x * block.y * block.z;
    // the runtime refuses launches of 2^32 lanes and more in a dimension
    if ((uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 || (uint64_t)grid.z * block.z >> 32)
        return set(hipErrorInvalidConfiguration);
    if (!g_fail.empty() && l.name.find(g_fail) != std::string::npos && g_fail_after-- <= 0)
        return set(hipErrorLaunchFailure);
    std::memset(l.arg, 0, sizeof l.arg);
    for (int i = 0; i < readable(l.name); ++i) std::memcpy(&l.arg[i], args[i], is_int(l.name, i) ? 4 : 8);
    g_log.push_back(l);
    if (!g_result.empty() && l.name.find("k_sum_partials") != std::string::npos) {
        for (const auto &h : g_host)
            if (l.arg[3] >= (uint64_t)h.first && l.arg[3] < (uint64_t)h.first + h.second)
                std::memcpy((void *)l.arg[3], g_result.data(), 8 * g_result.size());
        g_result.clear();
    }
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void *f, dim3 grid, dim3 block, void **args, unsigned shared, hipStream_t stream)
{
    return hipLaunchKernel(f, grid, block, args, shared, stream);
}
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    *p = (void *)(uintptr_t)0x7000000000ull;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;  // compute units
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    g_host.emplace_back((char *)*p, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *, size_t n, hipMemcpyKind k)
{
    if (k == hipMemcpyDeviceToHost) std::memset(dst, 0, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind k, hipStream_t)
{
    return hipMemcpy(dst, src, n, k);
}
// a stream that is being recorded cannot be waited for
hipError_t hipStreamSynchronize(hipStream_t) { return g_capturing ? set(hipErrorStreamCaptureUnsupported) : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = (hipEvent_t)1;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 8;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }

}  // extern "C"
