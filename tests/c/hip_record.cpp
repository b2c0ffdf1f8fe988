// The calls of the HIP runtime that the library makes, for a process without a device: nothing runs, and what is queued is kept as lines of
// text in the order of the calls ("launch <stream> <kernel> <dynamic LDS> <workgroups> <threads>", "record <stream> <event>", "wait <stream> <event>").
// Loaded with RTLD_GLOBAL ahead of the library, so that the library finds these. Device memory is addresses that nobody reads.
#include <stdint.h>
#include <stdio.h>

#include <map>
#include <string>

#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

static std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
static std::string g_log;
static uintptr_t g_next = 1ull << 40;
static struct {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_call;

static void line(const char* what, const void* stream, const void* event) {
    char text[96];
    snprintf(text, sizeof(text), "%s %zu %zu\n", what, (size_t)stream, (size_t)event);
    g_log += text;
}

extern "C" {
const char* hip_record_log() { return g_log.c_str(); }
void hip_record_clear() { g_log.clear(); }

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned int, void*, void*, void*, void*, int*) { names()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    g_call = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = g_call.grid, *block = g_call.block, *lds = g_call.lds, *stream = g_call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void**, size_t lds, hipStream_t stream) {
    char text[96];
    snprintf(text, sizeof(text), "launch %zu ", (size_t)stream);
    g_log += text + names()[kernel];
    snprintf(text, sizeof(text), " %zu %u %u\n", lds, grid.x * grid.y * grid.z, block.x);
    g_log += text;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* event, unsigned) {
    *event = (hipEvent_t)(g_next += 256);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t event, hipStream_t stream) {
    line("record", stream, event);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t event, unsigned) {
    line("wait", stream, event);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
    *p = (void*)g_next;
    g_next += (bytes + 511) / 256 * 256;
    return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* device) {
    *device = 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = (void*)(g_next += 256);
    return hipSuccess;
}
}
