// A HIP runtime for the CPU that records instead of launching: linked with the library's own objects it turns every
// public call into the list of kernels, grids and LDS sizes that the call would have launched, on a machine without a
// GPU.  Device memory is host memory (filled with 0xA5, so that what must be cleared shows), copies and memsets are
// performed, kernels never run.  Built and loaded by tests/test_routes_cpu.py.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {

struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
Config g_config;
std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> m;
    return m;
}
std::map<void*, size_t> g_blocks;
size_t g_last_block = 0, g_memset_bytes = 0;
hipError_t g_error = hipSuccess;   // of a launch, until it is asked for
std::string g_log;

}  // namespace

extern "C" {

// ---- what the tests read ----------------------------------------------------------------------------------------
// The launches since the last call, one "name gx gy gz threads lds" per line; the return value is the text's length.
size_t rec_take(char* buf, size_t n) {
    const size_t len = g_log.size();
    if (buf && n > len) std::memcpy(buf, g_log.c_str(), len + 1);
    if (buf) g_log.clear();
    return len;
}
size_t rec_last_block() { return g_last_block; }      // bytes of the last hipMalloc
size_t rec_held() {                                  // bytes held now
    size_t sum = 0;
    for (const auto& b : g_blocks) sum += b.second;
    return sum;
}
size_t rec_memset_bytes() { return g_memset_bytes; }  // bytes cleared by memsets so far

// ---- the runtime ------------------------------------------------------------------------------------------------
void** __hipRegisterFatBinary(const void*) {
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    g_config = Config{grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *lds = g_config.lds;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
    const auto it = kernels().find(fn);
    char line[512];
    std::snprintf(line, sizeof(line), "%s %u %u %u %u %zu\n", it == kernels().end() ? "?" : it->second.c_str(), grid.x, grid.y, grid.z, block.x, lds);
    g_log += line;
    // (what no launch may ask for)
    if (lds > 163840 || !grid.x || !grid.y || !grid.z || block.x * block.y * block.z > 1024) g_error = hipErrorInvalidConfiguration;
    return g_error;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::aligned_alloc(4096, (n + 4095) & ~(size_t)4095);
    if (!*p) return hipErrorOutOfMemory;
    std::memset(*p, 0xA5, n);
    g_blocks[*p] = n;
    g_last_block = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p && !g_blocks.erase(p)) return hipErrorInvalidValue;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
    std::memset(p, v, n);
    g_memset_bytes += n;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) { return hipMemcpy(d, s, n, kind); }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    alignas(256) static char place[256];
    *p = place;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = g_error;
    g_error = hipSuccess;
    return e;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}

}  // extern "C"
