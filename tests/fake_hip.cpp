// A HIP runtime for host tests, loaded before the library (RTLD_GLOBAL) so that its calls
// come here: no device, two pretended ones; every launch is recorded (fake_launches) and
// does nothing.  A stream of device d is the handle 0x1000 (d + 1); NULL is the current
// device's.
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
std::map<const void *, std::string> g_names;
std::string g_log, g_out;
Dim3 g_grid, g_block;
size_t g_lds;
void *g_stream;
int g_dev = 0, g_capturing = 0;
}  // namespace

extern "C" {
const char *fake_launches() {  // the launches since the last call, one per line
    g_out.swap(g_log);
    g_log.clear();
    return g_out.c_str();
}
void fake_capture(int on) { g_capturing = on; }

void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    g_names[host] = st == 0 ? d : name;
    free(d);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) {
    g_grid = grid, g_block = block, g_lds = lds, g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream) {
    *grid = g_grid, *block = g_block, *lds = g_lds, *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **, size_t lds, void *) {
    char line[64];
    snprintf(line, sizeof(line), " grid=%u,%u,%u block=%u lds=%zu\n", grid.x, grid.y, grid.z, block.x,
             lds);
    g_log += g_names[f] + line;
    return 0;
}
int hipGetDevice(int *d) { return *d = g_dev, 0; }
int hipSetDevice(int d) { return g_dev = d, 0; }
int hipStreamGetDevice(void *s, int *d) {
    *d = s ? (int)((uintptr_t)s / 0x1000) - 1 : g_dev;
    return 0;
}
int hipStreamIsCapturing(void *, int *status) { return *status = g_capturing, 0; }
int hipGetSymbolAddress(void **p, const void *) { return *p = (void *)(uintptr_t)(0x5000 + g_dev), 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "fake"; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipMalloc(void **p, size_t n) { return *p = malloc(n), 0; }
int hipFree(void *p) { return free(p), 0; }
int hipMemcpy(void *, const void *, size_t, int) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipMemcpyFromSymbol(void *d, const void *, size_t n, size_t, int) { return memset(d, 0, n), 0; }
int hipMemcpyToSymbol(const void *, const void *, size_t, size_t, int) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
}
