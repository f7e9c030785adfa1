// Stand-ins for the HIP runtime's calls (test infrastructure): libhzp's host code, that of kernels.hip included, linked with this file runs
// without a GPU.  Launches are recorded, not run; device memory is host memory; a call's status and the streams' capture status are what the test sets.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string kernel;
    unsigned grid[3], lds;
};

std::mutex mu;
std::vector<Launch> launches;
std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> names;      // (filled by the library's constructors)
    return names;
}
std::atomic<int> capture{0}, wait_status{0}, allocations{0};
std::atomic<long> host_allocations{-1};        // so many more succeed; negative: all do

}  // namespace

void *operator new(size_t bytes)
{
    if (host_allocations >= 0 && host_allocations-- == 0) {
        host_allocations = -1;
        throw std::bad_alloc();
    }
    if (void *const p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

// What the tests ask and set.
unsigned recorded() { return (unsigned)launches.size(); }
const char *recorded_kernel(unsigned i) { return launches[i].kernel.c_str(); }
void recorded_shape(unsigned i, unsigned *grid_and_lds)
{
    std::memcpy(grid_and_lds, launches[i].grid, sizeof launches[i].grid);
    grid_and_lds[3] = launches[i].lds;
}
void forget() { launches.clear(); }
void set_capture(int status) { capture = status; }
void set_wait_status(int status) { wait_status = status; }
int live_allocations() { return allocations; }
void fail_host_allocation(long which) { host_allocations = which; }
int host_allocation_failed() { return host_allocations.exchange(-1) < 0; }     // (and no further one fails)

void **__hipRegisterFatBinary(const void *)
{
    static void *handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    char *const text = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    kernels()[host] = text ? text : device;
    std::free(text);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipErrorInvalidConfiguration; }

hipError_t hipLaunchKernel(const void *function, dim3 grid, dim3, void **, size_t lds, hipStream_t)
{
    std::lock_guard<std::mutex> lock(mu);
    const auto known = kernels().find(function);
    if (known == kernels().end()) return hipErrorInvalidDeviceFunction;
    const long left = host_allocations.exchange(-1);        // (the record's own allocations succeed)
    launches.push_back({known->second, {grid.x, grid.y, grid.z}, (unsigned)lds});
    host_allocations = left;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status)
{
    *status = (hipStreamCaptureStatus)capture.load();
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "error set by the test"; }
hipError_t hipMalloc(void **out, size_t bytes)
{
    *out = std::malloc(bytes);
    if (*out) ++allocations;
    return *out ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    if (p) --allocations;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t bytes, hipMemcpyKind)
{
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }
hipError_t hipGetDevice(int *device)
{
    *device = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return (hipError_t)wait_status.load(); }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }       // no scheduler and no tuning here
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipErrorNotSupported; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventQuery(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipMemsetD32Async(hipDeviceptr_t, int, size_t, hipStream_t) { return hipErrorNotSupported; }

}  // extern "C"
