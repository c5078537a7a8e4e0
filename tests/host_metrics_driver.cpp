// Host-side driver for hodmas_image_metrics: the library's metrics source is
// linked with this file's HIP runtime, which launches nothing and whose pinned
// allocations fail as often as argv[1] says, each leaving its error for
// hipGetLastError as the real one does.  Exits 0 if the call returns argv[2].
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>

#include "hodmas.h"

namespace {
int failing = 0;
hipError_t last = hipSuccess;
hipError_t give(hipError_t e)
{
    if (e != hipSuccess)
        last = e;
    return e;
}
char device_memory[1 << 20];
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*)
{
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    *p = device_memory;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (failing-- > 0)
        return give(hipErrorOutOfMemory);
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void)
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
}

int main(int, char** argv)
{
    failing = std::atoi(argv[1]);
    const hodmas_rect r{0, 4, 0, 4};
    float image[16] = {};
    hodmas_metrics out;
    const hodmas_status first = hodmas_image_metrics(image, 4, 4, 1e-4, &r, &r, 16, nullptr, &out);
    const hodmas_status second = hodmas_image_metrics(image, 4, 4, 1e-4, &r, &r, 16, nullptr, &out);
    std::printf("%d, then %d\n", (int)first, (int)second);
    return first == std::atoi(argv[2]) && second == HODMAS_OK ? 0 : 1;
}
