// A HIP runtime that runs nothing: libgear.so's calls reach it instead of the
// installed one, and every kernel launch is handed to a callback.  Device memory is
// address ranges without storage, so calls on tables and batches of any size can
// be followed on the CPU.  Page-locked memory has a device address of its own,
// as memory that was locked after its allocation may have.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstring>
#include <map>
#include <string>

namespace {

constexpr uintptr_t kDeviceBase = 1ull << 44;
constexpr uintptr_t kLockedOffset = 1ull << 45;  // device address of locked memory - its host address

uintptr_t g_next = kDeviceBase;
std::map<uintptr_t, size_t> g_device, g_locked;  // base -> size
std::map<const void*, std::string> g_kernels;
hipError_t g_last = hipSuccess;
struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} g_config;
typedef void (*Callback)(const char* kernel, uint32_t grid, uint32_t block, void** args);
Callback g_callback = nullptr;
typedef void (*CopyCallback)(const void* dst, const void* src, uint64_t bytes);
CopyCallback g_copy = nullptr;

const std::pair<const uintptr_t, size_t>* range_of(const std::map<uintptr_t, size_t>& m, uintptr_t p) {
    auto it = m.upper_bound(p);
    if (it == m.begin()) return nullptr;
    --it;
    return p < it->first + it->second ? &*it : nullptr;
}

}  // namespace

extern "C" {

void stub_on_launch(Callback c) { g_callback = c; }
void stub_on_copy(CopyCallback c) { g_copy = c; }
void stub_lock(void* p, size_t bytes) { g_locked[(uintptr_t)p] = bytes; }
uint64_t stub_locked_offset() { return kLockedOffset; }

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
    g_kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    g_config = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *shared = g_config.shared;
    *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    // The limit of the launch calls: fewer than 2^32 work items.
    if ((uint64_t)grid.x * block.x > 0xFFFFFFFFull || grid.x == 0) return g_last = hipErrorInvalidConfiguration;
    if (g_callback) g_callback(g_kernels[f].c_str(), grid.x, block.x, args);
    return hipSuccess;
}

hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {  // a macro for the versioned name
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    return *s = hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)&g_last, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t bytes) {
    g_device[g_next] = bytes;
    *p = (void*)g_next;
    g_next += (bytes + 4095) / 4096 * 4096 + 4096;
    return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    void* m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    stub_lock(m, bytes);
    *p = m;
    return hipSuccess;
}
hipError_t hipHostFree(void*) { return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = (void*)((uintptr_t)h + kLockedOffset);
    return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) {
    if (g_copy) g_copy(dst, src, bytes);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, hipErrorInvalidValue; }

hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    std::memset(a, 0, sizeof(*a));
    const uintptr_t at = (uintptr_t)p;
    if (range_of(g_device, at)) {
        a->type = hipMemoryTypeDevice;
        a->devicePointer = (void*)at;
        return hipSuccess;
    }
    const bool host = range_of(g_locked, at) != nullptr;
    if (!host && !range_of(g_locked, at - kLockedOffset)) return g_last = hipErrorInvalidValue;
    a->type = hipMemoryTypeHost;
    a->hostPointer = (void*)(host ? at : at - kLockedOffset);
    a->devicePointer = (void*)(host ? at + kLockedOffset : at);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    const auto* r = range_of(g_device, (uintptr_t)p);
    if (r == nullptr) r = range_of(g_locked, (uintptr_t)p);
    if (r == nullptr) return g_last = hipErrorInvalidValue;
    *base = (hipDeviceptr_t)r->first;
    *size = r->second;
    return hipSuccess;
}

}  // extern "C"
