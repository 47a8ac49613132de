// Stands in for the HIP runtime: the library's host code runs to the end, nothing reaches a GPU, and every kernel launch is written
// down with its grid, its dynamic LDS and the cap on dynamic LDS that is in force for that kernel on the current device.
#include <cxxabi.h>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid, block;
    size_t lds, cap;
};
std::map<const void*, std::string> names;
std::map<std::pair<int, const void*>, size_t> caps;
std::vector<Launch> launches;
struct {
    Dim3 grid, block;
    size_t lds;
    void* stream;
} pending;
int device = 0, failing = 0, last_error = 0;
}  // namespace

extern "C" {

void rec_reset(int dev, int fail_attributes) {
    launches.clear();
    device = dev;
    failing = fail_attributes;
    last_error = 0;
}
int rec_count() { return (int)launches.size(); }
const char* rec_name(int i) { return launches[i].name.c_str(); }
void rec_shape(int i, uint32_t* grid, uint32_t* block, size_t* lds, size_t* cap) {
    const Launch& l = launches[i];
    grid[0] = l.grid.x; grid[1] = l.grid.y; grid[2] = l.grid.z;
    block[0] = l.block.x; block[1] = l.block.y; block[2] = l.block.z;
    *lds = l.lds;
    *cap = l.cap;
}

void** __hipRegisterFatBinary(const void*) {
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* mangled, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(mangled, nullptr, nullptr, &status);
    names[host] = plain && status == 0 ? plain : mangled;
    std::free(plain);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    pending = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = pending.grid;
    *block = pending.block;
    *lds = pending.lds;
    *stream = pending.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
    const auto cap = caps.find({device, f});
    launches.push_back({names[f], grid, block, lds, cap == caps.end() ? (size_t)64 * 1024 : cap->second});
    return 0;
}
int hipFuncSetAttribute(const void* f, int attribute, int value) {
    if (failing) return last_error = 1;
    if (attribute == 8) caps[{device, f}] = (size_t)value;      // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int hipGetDevice(int* d) {
    *d = device;
    return 0;
}
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipGetSymbolAddress(void** p, const void*) {
    *p = reinterpret_cast<void*>((uintptr_t)1 << 32);
    return 0;
}
int hipEventRecord(void*, void*) { return 0; }
}
