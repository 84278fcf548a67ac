// A HIP runtime for tests of libpf's host code: devices with an MI355X's
// numbers, host memory for device memory, launches recorded and not run.  Like
// the real one it refuses a launch that asks for more dynamic LDS than the
// kernel's limit on the current device (64 KB with its static LDS until
// hipFuncSetAttribute raises it).  Loaded before libpf under the runtime's
// soname.
#include <hip/hip_runtime_api.h>

#include <unistd.h>

#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>

namespace {

constexpr int kLds = 160 * 1024, kUnits = 256, kStatic = 256;
std::mutex mu;
thread_local int device = 0;
thread_local hipError_t last = hipSuccess;
int refuse_attr = 0, slow_attr_us = 0;
std::map<const void*, std::string> names;
std::map<std::pair<int, const void*>, int> limits;
struct Config {
    dim3 grid, block;
    size_t shm;
    hipStream_t stream;
};
thread_local Config pushed;
struct Launch {
    std::string name;
    unsigned grid, block;
    size_t lds;
};
thread_local Launch latest;
thread_local int launches = 0;

hipError_t result(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}

}  // namespace

extern "C" {

void stub_refuse_attributes(int on) { refuse_attr = on; }
void stub_slow_attributes(int us) { slow_attr_us = us; }
int stub_launches() { return launches; }
// The calling thread's latest accepted launch: kernel, workgroups, threads, dynamic LDS.
void stub_latest(char* name, int size, long long* out)
{
    std::strncpy(name, latest.name.c_str(), size - 1);
    out[0] = latest.grid;
    out[1] = latest.block;
    out[2] = (long long)latest.lds;
}

void** __hipRegisterFatBinary(const void*)
{
    static void* module;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*)
{
    names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shm, hipStream_t stream)
{
    pushed = {grid, block, shm, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shm, hipStream_t* stream)
{
    *grid = pushed.grid;
    *block = pushed.block;
    *shm = pushed.shm;
    *stream = pushed.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t shm, hipStream_t)
{
    std::lock_guard<std::mutex> lock(mu);
    const auto it = limits.find({device, f});
    const size_t limit = it == limits.end() ? 64 * 1024 - kStatic : it->second;
    if (shm > limit || !grid.x || !grid.y || !block.x) return result(hipErrorInvalidValue);
    latest = {names[f], grid.x, block.x, shm};
    ++launches;
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void* f, dim3 grid, dim3 block, void** args,
                                      unsigned shm, hipStream_t st)
{
    return hipLaunchKernel(f, grid, block, args, shm, st);
}
hipError_t hipGetDevice(int* d)
{
    *d = device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    device = d;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int)
{
    if (a == hipDeviceAttributeMaxSharedMemoryPerBlock) *v = kLds;
    else if (a == hipDeviceAttributeMultiprocessorCount) *v = kUnits;
    else return result(hipErrorInvalidValue);
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*)
{
    std::memset(a, 0, sizeof *a);
    a->sharedSizeBytes = kStatic;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v)
{
    if (slow_attr_us) usleep(slow_attr_us);
    if (refuse_attr || a != hipFuncAttributeMaxDynamicSharedMemorySize || v > kLds - kStatic)
        return result(hipErrorInvalidValue);
    std::lock_guard<std::mutex> lock(mu);
    limits[{device, f}] = v;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "refused by the stub"; }
hipError_t hipGetLastError(void)
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return result(hipErrorInvalidValue); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}

}  // extern "C"
