// Test aid: the part of the HIP runtime that the library calls, recorded instead of executed, so that what the host side
// launches (kernel, grid, LDS, on which device) can be looked at without a GPU. Loaded before the library, with its symbols
// global, into a process of its own. Nothing dereferences a device pointer here.
#include <cxxabi.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <utility>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Config { Dim3 grid, block; size_t lds; void* stream; };

int g_device = 0;
std::map<const void*, std::string> g_names;
std::map<std::pair<int, const void*>, int> g_lds_limit;  // requested per device
std::string g_log, g_kernels;
Config g_config;
void* g_modules[1];

int record(const void* f, Dim3 g, Dim3 b, size_t lds) {
    const auto limit = g_lds_limit.find({g_device, f});
    const bool allowed = lds <= 64 * 1024 || (limit != g_lds_limit.end() && lds <= (size_t)limit->second);
    g_log += g_names[f] + "\t" + std::to_string(g.x) + "\t" + std::to_string(g.y) + "\t" + std::to_string(g.z) + "\t" +
             std::to_string(b.x * b.y * b.z) + "\t" + std::to_string(lds) + "\t" + std::to_string(g_device) + "\t" +
             (allowed ? "1" : "0") + "\n";
    return 0;
}
}  // namespace

extern "C" {
char __hip_fatbin[1];  // for a library compiled for the host alone: there is no device code to point at
void recorder_set_device(int dev) { g_device = dev; }
void recorder_clear() { g_log.clear(); }
// One line per launch: kernel, grid x, y, z, threads, dynamic LDS bytes, device, whether that much LDS was asked for there.
const char* recorder_log() { return g_log.c_str(); }
// Every kernel of the library, one a line.
const char* recorder_kernels() { return g_kernels.c_str(); }

void** __hipRegisterFatBinary(const void*) { return g_modules; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    g_names[host] = status == 0 ? plain : name;
    std::free(plain);
    g_kernels += g_names[host] + "\n";
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    g_config = Config{grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*) { return record(f, grid, block, lds); }
int hipExtLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*, void*, void*, int) {
    return record(f, grid, block, lds);
}
int hipFuncSetAttribute(const void* f, int attr, int value) {
    if (attr == 8) g_lds_limit[{g_device, f}] = value;  // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int hipGetDevice(int* dev) { *dev = g_device; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = 256; return 0; }  // the only one asked for: compute units
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)(uintptr_t)0x7000000000; return 0; }
int hipGetLastError() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipEventCreate(void**) { return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }
}
