// A HIP runtime that records kernel launches instead of running them: loaded
// ahead of libbrownout_moe.so (global symbols), so that a test without a GPU
// sees which kernels a call launches, and with what grid, on a device whose
// answers the test chooses.
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

namespace {
struct Dim {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    uint32_t x, y, z;
};
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<Launch> launches;
Dim cfg_grid, cfg_block;
size_t cfg_shmem;
void* cfg_stream;
int g_device = 0, g_device_status = 0, g_cus = 256, g_cus_status = 0;
char g_array[1 << 21];
void* g_module;
}  // namespace

extern "C" {
void recorder_device(int device, int device_status, int cus, int cus_status) {
    g_device = device;
    g_device_status = device_status;
    g_cus = cus;
    g_cus_status = cus_status;
    launches.clear();
}
int recorder_count() { return (int)launches.size(); }
const char* recorder_name(int i) { return launches[i].name.c_str(); }
void recorder_grid(int i, uint32_t* g) {
    g[0] = launches[i].x;
    g[1] = launches[i].y;
    g[2] = launches[i].z;
}

int hipGetDevice(int* d) {
    *d = g_device;
    return g_device_status;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = g_cus;
    return g_cus_status;
}
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
    *p = g_array;
    return 0;
}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shmem, void* stream) {
    cfg_grid = g;
    cfg_block = b;
    cfg_shmem = shmem;
    cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* shmem, void** stream) {
    *g = cfg_grid;
    *b = cfg_block;
    *shmem = cfg_shmem;
    *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim, void**, size_t, void*) {
    launches.push_back({names()[f], g.x, g.y, g.z});
    return 0;
}
void** __hipRegisterFatBinary(const void*) { return &g_module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
    int status = 0;
    char* s = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    names()[host] = status == 0 && s ? s : device;
    free(s);
}
}
