// A stand-in for the HIP runtime that runs nothing: it records the launches,
// copies and attribute settings libsigk asks for, so that the host side's
// choices (kernel, grid, workspace) can be checked without a GPU.  Loaded in a
// process of its own before libsigk, under the runtime's soname.
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Event {
    std::string what, name;
    long long grid, block, lds;
};
std::map<const void*, std::string> g_names;
std::map<std::string, int> g_occ;
std::vector<Event> g_events;
int g_cus = 256;
struct Dim3 {
    uint32_t x, y, z;
};
std::vector<std::string> g_cfg;
std::string name_of(const void* f) {
    auto it = g_names.find(f);
    return it == g_names.end() ? "?" : it->second;
}
struct Config {
    Dim3 grid, block;
    size_t lds;
    void* stream;
} g_config;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned,
                           void*, void*, void*, void*, int*) {
    g_names[host] = device_name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void* s) {
    g_config = {g, b, lds, s};
    return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* lds, void** s) {
    *g = g_config.grid;
    *b = g_config.block;
    *lds = g_config.lds;
    *s = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void**, size_t lds, void*) {
    g_events.push_back({"launch", name_of(f), (long long)g.x * g.y * g.z, (long long)b.x, (long long)lds});
    return 0;
}
int hipFuncSetAttribute(const void* f, int, int value) {
    g_events.push_back({"attribute", name_of(f), 0, 0, value});
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds) {
    const std::string name = name_of(f);
    *n = 4;  // waves per CU
    size_t best = 0;
    for (auto& o : g_occ)
        if (o.first.size() > best && name.find(o.first) != std::string::npos) {
            best = o.first.size();
            *n = o.second;
        }
    *n /= block / 64;
    if (lds > 0 && *n > (int)(163840 / lds)) *n = (int)(163840 / lds);
    return 0;
}
int hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = g_cus;
    return 0;
}
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "recorded"; }
int hipGetSymbolAddress(void** p, const void*) {
    *p = (void*)(uintptr_t)0x10000000000ull;
    return 0;
}
int hipMemcpyAsync(void*, const void*, size_t n, int, void*) {
    g_events.push_back({"copy", "", 0, 0, (long long)n});
    return 0;
}
int hipStreamSynchronize(void*) {
    g_events.push_back({"wait", "", 0, 0, 0});
    return 0;
}

void rec_set_cus(int n) { g_cus = n; }
void rec_set_occupancy(const char* part, int n) { g_occ[part] = n; }
void rec_clear() { g_events.clear(); }
int rec_count() { return (int)g_events.size(); }
const char* rec_what(int i) { return g_events[(size_t)i].what.c_str(); }
const char* rec_name(int i) { return g_events[(size_t)i].name.c_str(); }
void rec_sizes(int i, long long* out) {
    const Event& e = g_events[(size_t)i];
    out[0] = e.grid;
    out[1] = e.block;
    out[2] = e.lds;
}
}
