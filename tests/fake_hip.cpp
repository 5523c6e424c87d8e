// A HIP runtime without a device, for CPU tests of the library's host code: loaded
// before libpvdock.so, its functions take the place of libamdhip64's.  Memory is
// host memory, kernels are recorded instead of run, and the documented rules that
// the tests are about hold: a failing call leaves its error for hipGetLastError,
// a launch of 2^32 threads or more in a dimension is refused, hipFree waits for
// the device, and a device may run out of memory.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};

thread_local hipError_t g_last = hipSuccess;
thread_local int g_device = 0;
thread_local struct { dim3 grid, block; size_t lds; hipStream_t stream; } g_config;
std::map<const void*, std::string> g_names;
std::map<void*, size_t> g_blocks;
std::vector<Launch> g_launches;
size_t g_used = 0, g_limit = (size_t)1 << 60;
int g_syncs = 0, g_capturing = 0, g_handles = 0;

hipError_t ret(hipError_t e)
{
    if (e != hipSuccess) g_last = e;
    return e;
}
template <class H>
hipError_t handle(H* h) { *h = (H)(uintptr_t)(0x1000 + 16 * ++g_handles); return hipSuccess; }

}  // namespace

extern "C" {

// ---------------------------------------------------------------- the tests' side
void fake_memory(size_t limit) { g_limit = limit; }
size_t fake_used() { return g_used; }
int fake_device_syncs() { return g_syncs; }
void fake_capture(int on) { g_capturing = on; }
int fake_current_device() { return g_device; }
int fake_launches() { return (int)g_launches.size(); }
void fake_clear() { g_launches.clear(); }
// grid, block (x, y, z each), LDS bytes and stream of launch i; its kernel's name
const char* fake_launch(int i, uint64_t v[8])
{
    const Launch& k = g_launches[i];
    const uint64_t w[8] = {k.grid.x, k.grid.y, k.grid.z, k.block.x, k.block.y, k.block.z, k.lds, (uint64_t)(uintptr_t)k.stream};
    std::memcpy(v, w, sizeof(w));
    return k.name.c_str();
}

// ---------------------------------------------------------------- the runtime's side
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : e == hipSuccess ? "no error" : "error"; }
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n)
{
    *p = nullptr;
    if (g_capturing) return ret(hipErrorStreamCaptureUnsupported);
    if (g_used + n > g_limit) return ret(hipErrorOutOfMemory);
    void* m = mmap(nullptr, std::max<size_t>(n, 1), PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return ret(hipErrorOutOfMemory);
    g_blocks[m] = n;
    g_used += n;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (!p) return hipSuccess;
    if (g_capturing) return ret(hipErrorStreamCaptureUnsupported);
    auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return ret(hipErrorInvalidDevicePointer);
    munmap(p, std::max<size_t>(it->second, 1));
    g_used -= it->second;
    g_blocks.erase(it);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    ++g_syncs;
    return g_capturing ? ret(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = mmap(nullptr, (size_t)64 << 20, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return handle(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return handle(g); }
hipError_t hipEventCreate(hipEvent_t* e) { return handle(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return handle(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) { return handle(x); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    g_config = {g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s)
{
    *g = g_config.grid; *b = g_config.block; *lds = g_config.lds; *s = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t s)
{
    const uint64_t lim = (uint64_t)1 << 32;
    if (!g.x || !g.y || !g.z || (uint64_t)g.x * b.x >= lim || (uint64_t)g.y * b.y >= lim || (uint64_t)g.z * b.z >= lim ||
        b.x * b.y * b.z > 1024 || lds > 160 * 1024)
        return ret(hipErrorInvalidConfiguration);
    g_launches.push_back({g_names[f], g, b, lds, s});
    return hipSuccess;
}
// 160 KB of LDS and the waves the kernels' registers allow: eight per CU, twelve
// for the dock and optimisation kernels built for three waves per SIMD (team
// size 0, 2 or 4 as the last template argument)
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int threads, size_t lds)
{
    const std::string& k = g_names[f];
    auto ends = [&](const char* t) { return k.find(t) != std::string::npos; };
    const bool three = (ends("dock_kernel") || ends("local_opt")) && (ends("ELi0EE") || ends("ELi2EE") || ends("ELi4EE"));
    const int waves = (threads + 63) / 64;
    *n = std::min<int>((three ? 12 : 8) / waves, (int)(160 * 1024 / std::max<size_t>(lds, 1)));
    return hipSuccess;
}

}  // extern "C"
