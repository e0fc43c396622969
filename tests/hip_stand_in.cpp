// A stand-in for the HIP runtime on a machine without a GPU: libfr.so's host
// code runs against it, kernels are logged instead of run and take a time
// given by their name.  Loaded before libfr.so with global symbols, so that
// libfr.so binds to it.
//
// Device memory is host memory, events read a simulated clock, and a kernel's
// dynamic LDS limit is 64 KiB on each device until hipFuncSetAttribute raises
// it there for that kernel.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <regex>
#include <string>
#include <utility>
#include <vector>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
struct Config {
    Dim3 grid, block;
    size_t lds;
    void *stream;
};
struct State {
    int device = 0;
    double clock = 0;                                    // microseconds
    std::vector<Config> configs;
    std::map<const void *, std::string> names;           // host function -> kernel
    std::map<std::pair<int, const void *>, int> lds_limit;
    std::vector<std::pair<std::regex, double>> costs;    // of the names that match, microseconds
    std::vector<std::pair<std::regex, double>> cold;     // and after another kernel (caches)
    const void *last = nullptr;
    std::string log;                                     // "device grid name" per launch
    std::map<const void *, void *> symbols;
};
State &S() {
    static State s;
    return s;
}
constexpr int INVALID_VALUE = 1;
}  // namespace

extern "C" {
// ---- control ----
void stand_in_device(int d) { S().device = d; }
void stand_in_cost(const char *name, double us) { S().costs.emplace_back(std::regex(name), us); }
void stand_in_cold(const char *name, double us) { S().cold.emplace_back(std::regex(name), us); }
void stand_in_clear() {
    S().costs.clear();
    S().cold.clear();
    S().log.clear();
}
const char *stand_in_log() { return S().log.c_str(); }

// ---- registration and launches ----
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
    S().names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *stream) {
    S().configs.push_back({g, b, lds, stream});
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **stream) {
    const Config c = S().configs.back();
    S().configs.pop_back();
    *g = c.grid;
    *b = c.block;
    *lds = c.lds;
    *stream = c.stream;
    return 0;
}
static int g_error = 0;
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **, size_t lds, void *) {
    State &s = S();
    const auto lim = s.lds_limit.find({s.device, f});
    if (lds > size_t(lim == s.lds_limit.end() ? 65536 : lim->second)) return g_error = INVALID_VALUE;
    const std::string &name = s.names[f];
    s.log += std::to_string(s.device) + " " + std::to_string(grid.x) + " " + name + "\n";
    double us = 1;
    for (const auto &c : s.costs)
        if (std::regex_search(name, c.first)) us += c.second;
    if (f != s.last)
        for (const auto &c : s.cold)
            if (std::regex_search(name, c.first)) us += c.second;
    s.last = f;
    s.clock += us;
    return 0;
}
int hipFuncSetAttribute(const void *f, int attr, int value) {
    if (attr == 8) S().lds_limit[{S().device, f}] = value;   // MaxDynamicSharedMemorySize
    return 0;
}
int hipGetLastError() {
    const int e = g_error;
    g_error = 0;
    return e;
}
const char *hipGetErrorString(int) { return "stand-in error"; }

// ---- devices, memory ----
int hipGetDevice(int *d) {
    *d = S().device;
    return 0;
}
int hipDeviceGetAttribute(int *v, int, int) {
    *v = 256;
    return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void **p, size_t n) {
    *p = std::aligned_alloc(256, (n + 511) / 256 * 256);
    std::memset(*p, 0, n);
    return 0;
}
int hipFree(void *p) {
    std::free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int, void *) {
    for (size_t i = 0; i < h; ++i) std::memcpy(static_cast<char *>(d) + i * dp, static_cast<const char *>(s) + i * sp, w);
    return 0;
}
int hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *) {
    std::memset(d, v, n);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *sym) {
    void *&q = S().symbols[sym];
    if (!q) q = std::calloc(1, 1 << 20);
    *p = q;
    return 0;
}

// ---- events, streams ----
int hipEventCreateWithFlags(void **e, unsigned) {
    *e = new double(0);
    return 0;
}
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *e) {
    delete static_cast<double *>(e);
    return 0;
}
int hipEventRecord(void *e, void *) {
    *static_cast<double *>(e) = S().clock;
    return 0;
}
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) {
    *ms = float((*static_cast<double *>(b) - *static_cast<double *>(a)) * 1e-3);
    return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned) {
    *s = std::malloc(1);
    return 0;
}
int hipStreamDestroy(void *s) {
    std::free(s);
    return 0;
}
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
}
