// A HIP runtime without a GPU for host-side tests: memory is host memory, a launch only
// calls back (name, grid, LDS bytes, device, arguments), streams name a device.  Loaded
// ahead of libcgs.so with its symbols global, so the library binds to it.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>

namespace {
using Callback = void (*)(const char* name, const unsigned* grid, size_t lds, int device, void** args);
Callback g_call = nullptr;
int g_current = 0, g_attributes = 1;
hipError_t g_error = hipSuccess;
std::map<const void*, std::string> g_names;
std::map<std::pair<const void*, int>, int> g_dynamic;   // (kernel, device): LDS beyond 64 KB allowed
constexpr size_t kStatic = 512;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_config;
int device_of(hipStream_t s) { return s ? *reinterpret_cast<int*>(s) : g_current; }
alignas(256) unsigned char g_array[32 << 20];
}  // namespace

extern "C" {
void fake_callback(Callback f) { g_call = f; }
void fake_set_device(int d) { g_current = d; }
void fake_func_attributes(int on) { g_attributes = on; }   // 0: hipFuncGetAttributes fails
void* fake_stream(int device) { return new int(device); }

void** __hipRegisterFatBinary(const void*) { return new void*(nullptr); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    g_names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    g_config = {g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
    *g = g_config.grid;
    *b = g_config.block;
    *lds = g_config.lds;
    *s = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void** args, size_t lds, hipStream_t s) {
    const unsigned grid[3] = {g.x, g.y, g.z};
    const auto it = g_dynamic.find({f, device_of(s)});
    if (lds + kStatic > 65536 && (it == g_dynamic.end() || (size_t)it->second < lds))
        return g_error = hipErrorInvalidValue;
    if (g_call) g_call(g_names[f].c_str(), grid, lds, device_of(s), args);
    return hipSuccess;
}

hipError_t hipGetDevice(int* d) { return *d = g_current, hipSuccess; }
hipError_t hipSetDevice(int d) { return g_current = d, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { return *d = device_of(s), hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 << 10 : 0;
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
    std::memset(a, 0, sizeof *a);
    a->sharedSizeBytes = kStatic;
    return g_attributes ? hipSuccess : hipErrorInvalidDeviceFunction;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) {
    return g_dynamic[{f, g_current}] = v, hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_error;
    return g_error = hipSuccess, e;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = g_array, hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t*, const void*) { return hipErrorInvalidValue; }

hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }

hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)&g_config, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)new int(g_current), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}
