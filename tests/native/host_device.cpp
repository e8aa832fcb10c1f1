// A stand-in for the device runtime, for tests of the library's host side on a
// machine without a GPU: "device" memory is zeroed host memory, copies are
// memcpy, kernels are recorded (name, grid) and not run, and the time between
// two events is the sum of the launches' costs set by the test.  Loaded before
// the library with global symbols (tests/test_host_launch.py).
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {
struct Dim { uint32_t x, y, z; };
struct Config { Dim grid, block; size_t shared; void *stream; } g_config;
std::map<const void *, std::string> g_kernels;
std::map<std::string, long> g_best, g_grid;    // kernel name part: cheapest grid; kernel name: last grid
std::set<void *> g_live;
double g_clock = 0.0;
long g_fail_in = -1;                            // device allocations until one fails (-1: none)
long g_bad = 0;                                 // memory freed twice, copies to or from nowhere
struct Event { double t = 0.0; };
constexpr int OK = 0, INVALID = 1, NO_MEMORY = 2;
int copy(void *d, const void *s, size_t n) {
    if (n && (!d || !s)) { ++g_bad; return INVALID; }
    if (n) std::memmove(d, s, n);
    return OK;
}
}  // namespace

extern "C" {
// ---- controls
void host_device_fail_in(long n) { g_fail_in = n; }
// launches of kernels whose name holds `part` cost 1 + the relative distance of their grid from `grid`
void host_device_best_grid(const char *part, long grid) { g_best[part] = grid; }
long host_device_last_grid(const char *part) {
    for (auto &k : g_grid)
        if (k.first.find(part) != std::string::npos) return k.second;
    return -1;
}
void host_device_forget() { g_grid.clear(); }
long host_device_live() { return (long)g_live.size(); }
long host_device_bad() { return g_bad; }

// ---- module registration and launches
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    g_kernels[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shared, void *stream) {
    g_config = Config{grid, block, shared, stream};
    return OK;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *shared, void **stream) {
    *grid = g_config.grid; *block = g_config.block; *shared = g_config.shared; *stream = g_config.stream;
    return OK;
}
int hipLaunchKernel(const void *f, Dim grid, Dim, void **, size_t, void *) {
    const std::string &name = g_kernels[f];
    const long n = (long)grid.x * grid.y * grid.z;
    if (n == 0) return INVALID;
    g_grid[name] = n;
    double cost = 0.0;
    for (auto &b : g_best)
        if (name.find(b.first) != std::string::npos) cost = 1.0 + (n > b.second ? n - b.second : b.second - n) / (double)b.second;
    g_clock += cost;
    return OK;
}

// ---- memory
int hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (g_fail_in >= 0 && g_fail_in-- == 0) return NO_MEMORY;
    *p = std::calloc(1, n ? n : 1);
    if (!*p) return NO_MEMORY;
    g_live.insert(*p);
    return OK;
}
int hipFree(void *p) {
    if (p && !g_live.erase(p)) { ++g_bad; return INVALID; }
    std::free(p);
    return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n ? n : 1); return *p ? OK : NO_MEMORY; }
int hipHostFree(void *p) { std::free(p); return OK; }
int hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return OK; }
int hipMemcpy(void *d, const void *s, size_t n, int) { return copy(d, s, n); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return copy(d, s, n); }
int hipMemcpy2D(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int) {
    for (size_t r = 0; r < h; ++r) std::memmove((char *)d + r * dp, (const char *)s + r * sp, w);
    return OK;
}
int hipMemset(void *d, int v, size_t n) { if (n) std::memset(d, v, n); return OK; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { if (n) std::memset(d, v, n); return OK; }
int hipPointerGetAttributes(void *, const void *) { return INVALID; }   // (host pointers)
int hipGetSymbolAddress(void **p, const void *) { static double a[8]; *p = a; return OK; }

// ---- device, streams, events
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return OK; }
int hipDeviceSynchronize() { return OK; }
int hipFuncSetAttribute(const void *, int, int) { return OK; }
int hipGetLastError() { return OK; }
const char *hipGetErrorString(int e) { return e == NO_MEMORY ? "out of memory" : "invalid value"; }
int hipStreamCreateWithFlags(void **s, unsigned) { static char c; *s = &c; return OK; }
int hipStreamDestroy(void *) { return OK; }
int hipStreamSynchronize(void *) { return OK; }
int hipEventCreate(void **e) { *e = new Event; return OK; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = new Event; return OK; }
int hipEventDestroy(void *e) { delete (Event *)e; return OK; }
int hipEventRecord(void *e, void *) { ((Event *)e)->t = g_clock; return OK; }
int hipEventSynchronize(void *) { return OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = (float)(((Event *)b)->t - ((Event *)a)->t); return OK; }
int hipStreamBeginCapture(void *, int) { return INVALID; }
int hipStreamEndCapture(void *, void **) { return INVALID; }
int hipGraphInstantiate(void **, void *, void *, char *, size_t) { return INVALID; }
int hipGraphLaunch(void *, void *) { return INVALID; }
int hipGraphDestroy(void *) { return INVALID; }
int hipGraphExecDestroy(void *) { return INVALID; }
}
