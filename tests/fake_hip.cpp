// A stand-in for the HIP runtime calls that liboif.so makes, for tests of its host code without a GPU: two devices
// whose memory is host memory, no kernel run but the one that hands results to the host.  It enforces what the real
// one does about devices: a kernel launch needs the stream's device current, an event belongs to the device it was
// created on.  Loaded ahead of the real runtime with RTLD_GLOBAL.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

struct ihipStream_t { int device; };
struct ihipEvent_t { int device; };

namespace {
thread_local int current = 0;
std::map<const void*, std::string> kernels;
std::map<std::string, unsigned> blocks;  // of each kernel's last launch
std::map<const void*, char*> vars;
hipError_t get(void** p, size_t n) {
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256 + 256);
    if (!*p) return hipErrorOutOfMemory;
    std::memset(*p, 0, n);
    return hipSuccess;
}
hipError_t event(hipEvent_t* e) {
    *e = new ihipEvent_t{current};
    return hipSuccess;
}
struct Gather {  // GatherSrc of oif_device.h
    const void* p[3];
    unsigned n[3];
};
}  // namespace

extern "C" {
int fake_current() { return current; }
void fake_set_current(int d) { current = d; }
unsigned fake_blocks(const char* part_of_name) {
    for (const auto& b : blocks)
        if (b.first.find(part_of_name) != std::string::npos) return b.second;
    return 0;
}

hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = new ihipStream_t{current}; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return event(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return event(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    return e->device == s->device ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return get(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return get(p, n); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

// the kernels' host stubs: launch configuration, then hipLaunchKernel
static thread_local dim3 grid, block;
static thread_local size_t shared;
static thread_local hipStream_t on;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
    grid = g, block = b, shared = sh, on = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s) {
    *g = grid, *b = block, *sh = shared, *s = on;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return (void**)std::malloc(8); }
void __hipUnregisterFatBinary(void** p) { std::free(p); }
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { vars[var] = (char*)std::calloc(size, 1); }
hipError_t hipGetSymbolAddress(void** p, const void* sym) {
    *p = vars[sym];
    return *p ? hipSuccess : hipErrorInvalidSymbol;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void** args, size_t, hipStream_t s) {
    if (s && s->device != current) return hipErrorInvalidHandle;
    blocks[kernels[f]] = g.x;
    if (kernels[f].find("GatherSrc") != std::string::npos) {
        const Gather& g = *(const Gather*)args[0];
        char* dst = *(char**)args[1];
        for (int a = 0; a < 3; ++a) {
            if (g.n[a]) std::memcpy(dst, g.p[a], 4 * (size_t)g.n[a]);
            dst += 4 * (size_t)g.n[a];
        }
    }
    return hipSuccess;
}
}
