// Stand-ins for the HIP calls of a run's host side (tests/launches.py): no
// device work, every launch recorded by its kernel's name and launch shape.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <dlfcn.h>

#include <cstring>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string name;
    unsigned grid, block;
    size_t lds;
};
std::vector<Launch> launches;
int fail_at = -1;
struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} pushed;
}  // namespace

extern "C" {

// launch number `at` (from 0) returns an error; -1: none
void recorder_reset(int at) {
    launches.clear();
    fail_at = at;
}
int recorder_count() { return (int)launches.size(); }
const char *recorder_get(int i, unsigned *grid, unsigned *block, size_t *lds) {
    *grid = launches[i].grid;
    *block = launches[i].block;
    *lds = launches[i].lds;
    return launches[i].name.c_str();
}

hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **, size_t lds, hipStream_t) {
    Dl_info info;
    const bool found = dladdr(fn, &info) && info.dli_sname && info.dli_saddr == fn;
    const int n = (int)launches.size();
    launches.push_back({found ? info.dli_sname : "", grid.x * grid.y * grid.z, block.x, lds});
    return n == fail_at ? hipErrorLaunchFailure : hipSuccess;
}
// kernel<<<>>> is these two and a launch
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    pushed = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
    *grid = pushed.grid;
    *block = pushed.block;
    *lds = pushed.lds;
    *stream = pushed.stream;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(to, from, n);   // "device" memory of these runs is host memory
    return hipSuccess;
}

}  // extern "C"
