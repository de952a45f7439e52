// A stand-in for the HIP host API the library calls, so that its host
// bookkeeping runs without a GPU: "device" memory is host memory, kernels do
// nothing but are counted by name, and a call can be made to fail.  Loaded
// with RTLD_GLOBAL ahead of the library, whose references it then satisfies.
#include <hip/hip_runtime.h>

#include <dlfcn.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::map<void *, size_t> allocs;    // hipMalloc
std::vector<size_t> pool_allocs;    // hipMallocFromPoolAsync, in call order
std::vector<std::string> kernels;   // in launch order
std::vector<int64_t> grids;         // their workgroups
dim3 pushed_grid, pushed_block;     // of the launch being configured
int fail_records = 0;               // the next event records fail
std::string fast_kernel;            // launches timed as twice as fast
int stream_syncs = 0;
unsigned char symbol[1 << 20];
}  // namespace

extern "C" {

// what the tests read and set
int64_t fake_device_bytes()
{
    int64_t n = 0;
    for (const auto &a : allocs) n += (int64_t)a.second;
    return n;
}
int64_t fake_pool_allocs() { return (int64_t)pool_allocs.size(); }
int64_t fake_pool_bytes(int64_t k) { return (int64_t)pool_allocs[(size_t)k]; }
int64_t fake_launches(const char *part)
{
    int64_t n = 0;
    for (const auto &k : kernels) n += k.find(part) != std::string::npos;
    return n;
}
int64_t fake_workgroups(const char *part)   // of the last such launch
{
    for (size_t k = kernels.size(); k-- > 0;)
        if (kernels[k].find(part) != std::string::npos) return grids[k];
    return -1;
}
void fake_fail_records(int n) { fail_records = n; }
void fake_fast_kernel(const char *part) { fast_kernel = part; }
int fake_stream_syncs() { return stream_syncs; }
void fake_clear()
{
    pool_allocs.clear();
    kernels.clear();
    grids.clear();
    stream_syncs = 0;
}

hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = symbol, hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::calloc(1, n);
    allocs[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    allocs.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *)
{
    *p = reinterpret_cast<hipMemPool_t>(symbol);
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t, hipStream_t)
{
    pool_allocs.push_back(n);
    *p = std::malloc(64);   // nothing reads it
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t) { return std::free(p), hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    return std::memcpy(d, s, n), hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t *e) { return *e = reinterpret_cast<hipEvent_t>(symbol), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t)
{
    if (fail_records > 0) return --fail_records, hipErrorUnknown;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    const bool fast = !fast_kernel.empty() && !kernels.empty() && kernels.back().find(fast_kernel) != std::string::npos;
    *ms = fast ? 0.5f : 1.0f;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    return *s = hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return ++stream_syncs, hipSuccess; }

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    pushed_grid = grid;
    pushed_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream)
{
    *grid = pushed_grid;
    *block = pushed_block;
    *lds = 0;
    *stream = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **, size_t, hipStream_t)
{
    Dl_info info;
    kernels.push_back(dladdr(f, &info) && info.dli_sname ? info.dli_sname : "?");
    grids.push_back((int64_t)grid.x * grid.y * grid.z);
    return hipSuccess;
}
}
