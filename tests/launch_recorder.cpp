// A HIP runtime that launches nothing and writes down what it was asked to launch, for tests of the launch rules on a
// machine without a GPU (tests/launch_shapes.py).  It holds just the calls libkvc.so makes and is loaded in the place of
// libamdhip64.so.7.
#include "kvc_common.h"

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
    std::string kernel;  // mangled
    dim3 grid, block;
    size_t lds;  // beside the kernel's own
    unsigned long long line;  // where in the pool the encoder ends to keep payloads in the last-level cache, or the decoder begins to read past it; bytes
};
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<Launch>& launches() {
    static std::vector<Launch> v;
    return v;
}
hipMemoryType pool_type = hipMemoryTypeDevice;
int pool_device = 0;
}  // namespace

extern "C" {
void rec_clear() { launches().clear(); }
int rec_count() { return (int)launches().size(); }
const char* rec_kernel(int i) { return launches()[i].kernel.c_str(); }
void rec_shape(int i, unsigned* grid, unsigned* block, unsigned* lds) {
    *grid = launches()[i].grid.x;
    *block = launches()[i].block.x;
    *lds = (unsigned)launches()[i].lds;
}
unsigned long long rec_line(int i) { return launches()[i].line; }
void rec_memory(int type, int device) { pool_type = (hipMemoryType)type, pool_device = device; }  // what every address is from now on

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned int, void*, void*, dim3*, dim3*, int*) { names()[host] = device; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipErrorInvalidValue; }

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
    const std::string& name = names().at(f);
    unsigned long long line = 0;
    if (name.find("10k_compressI") != std::string::npos) line = static_cast<const kvc::EncodeArgs*>(args[0])->kept_units * 16;
    if (name.find("12k_decompressI") != std::string::npos) line = static_cast<const kvc::DecodeArgs*>(args[0])->near_bytes;
    launches().push_back({name, grid, block, lds, line});
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t) {
    *n = threads == 1024 ? 1 : 4;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipMalloc(void** p, size_t n) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { return memset(p, v, n), hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = const_cast<void*>(s), hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof *a);
    a->type = pool_type;
    a->device = pool_device;
    a->devicePointer = const_cast<void*>(p);
    return hipSuccess;
}
}
