// Test-only: sqrt_normal against the library's square root and against the
// float64 root rounded once, for every float of a range of bit patterns.
#include <hip/hip_runtime.h>

#include "device_common.h"

__global__ void check_kernel(unsigned lo, unsigned n, unsigned long long *differ) {
    unsigned long long bad_lib = 0, bad_exact = 0;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float x = __uint_as_float(lo + i);
        const unsigned s = __float_as_uint(restore::sqrt_normal(x));
        bad_lib += s != __float_as_uint(sqrtf(x));
        bad_exact += s != __float_as_uint((float)sqrt((double)x));
    }
    if (bad_lib) atomicAdd(differ, bad_lib);
    if (bad_exact) atomicAdd(differ + 1, bad_exact);
}

// bit patterns lo .. lo + n - 1; differ: two zeroed counters on the device
extern "C" int check_sqrt_normal(unsigned lo, unsigned n, unsigned long long *differ, void *stream) {
    if (n == 0 || n > 0x7fffffffu) return -1;
    unsigned long long *p = differ;
    void *args[] = {&lo, &n, &p};
    return (int)hipLaunchKernel((const void *)check_kernel, dim3(4096), dim3(256), args, 0,
                                static_cast<hipStream_t>(stream));
}
