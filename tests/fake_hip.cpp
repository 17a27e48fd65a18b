// A HIP runtime of the host, preloaded by test_create_host.py: memory is the host's, kernels do nothing, and an allocation of
// FAKE_HIP_REFUSE_FROM bytes or more (up to FAKE_HIP_REFUSE_TO) is refused and leaves its error behind as HIP does. Launches are noted
// down: fake_hip_take_launches gives "mangled name, grid x, grid y, bytes of dynamic LDS" a line, and forgets them.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

static hipError_t last = hipSuccess;
static char symbol[64];
static struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} config;

static std::map<const void*, std::string>& kernels() {      // registered before this file's static objects are made
    static std::map<const void*, std::string> k;
    return k;
}
static std::string launches;

static long long limit(const char* name, long long otherwise) {
    const char* v = getenv(name);
    return v ? atoll(v) : otherwise;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if ((long long)n >= limit("FAKE_HIP_REFUSE_FROM", 1LL << 62) && (long long)n <= limit("FAKE_HIP_REFUSE_TO", 1LL << 62)) return last = hipErrorOutOfMemory;
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    return *p ? hipSuccess : (last = hipErrorOutOfMemory);
}
hipError_t hipFree(void* p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels()[stub] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    config = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* stub, dim3 grid, dim3, void**, size_t lds, hipStream_t) {
    launches += kernels()[stub] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + " " + std::to_string(lds) + "\n";
    return hipSuccess;
}
const char* fake_hip_take_launches(void) {
    static std::string taken;
    taken.swap(launches);
    launches.clear();
    return taken.c_str();
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = symbol;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
}
