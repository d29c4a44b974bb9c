// The few HIP runtime functions librac.so calls, as stand-ins that run nothing
// and write down each launch: loaded ahead of librac.so (RTLD_GLOBAL), they
// take the place of the runtime's, so the kernels a call would launch can be
// seen on a machine without a GPU.  The device they describe has 256 compute
// units that hold 32 wavefronts each (no kernel limited by registers or LDS).
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::string g_log;
char g_symbol[1 << 20];
struct Dim {
    unsigned x, y, z;
};
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    names()[host] = name;
}
int hipGetDevice(int* dev) { return *dev = 0; }
int hipDeviceGetAttribute(int* v, int, int) {
    *v = 256;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t) {
    *n = 32 / (threads / 64);
    return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
    *p = g_symbol;
    return 0;
}
int hipMemcpyAsync(void* dst, const void*, size_t n, int, void*) {  // (copies to the host only)
    memset(dst, 0, n);
    return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipLaunchKernel(const void* f, Dim grid, Dim block, void**, size_t lds, void*) {
    char line[96];
    snprintf(line, sizeof line, "\t%u\t%u\t%u\t%zu\n", grid.x, grid.y, block.x, lds);
    const auto it = names().find(f);
    g_log += (it == names().end() ? "?" : it->second) + line;
    return 0;
}
const char* recorded() { return g_log.c_str(); }
void forget() { g_log.clear(); }
const char* registered() {  // every kernel of the library, a line each
    static std::string all;
    all.clear();
    for (const auto& n : names()) all += n.second + "\t0\t0\t0\t0\n";
    return all.c_str();
}
}
