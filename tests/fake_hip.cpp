// A stand-in for the HIP runtime that runs no kernel: memory is the host's,
// launches are counted by kernel name, and allocations can be made to fail.
// Loaded before libsv.so, whose calls it then takes, in processes that test
// the host code without a device.
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

struct dim3_ { unsigned x, y, z; };

static std::map<const void *, std::string> g_names;
static std::map<std::string, long> g_launches;
static std::set<void *> g_live; // allocations not freed yet
static size_t g_limit = ~(size_t)0; // largest allocation that succeeds

static int take(void **p, size_t bytes) {
    if (bytes > g_limit) return 2; // out of memory
    *p = std::malloc(bytes);
    if (!*p) return 2;
    g_live.insert(*p);
    return 0;
}
static int give(void *p) {
    if (p && !g_live.erase(p)) return 1;
    std::free(p);
    return 0;
}

extern "C" {
void fake_limit(size_t bytes) { g_limit = bytes; }
long fake_live() { return (long)g_live.size(); }
long fake_launches(const char *part) {
    long n = 0;
    for (const auto &e : g_launches)
        if (e.first.find(part) != std::string::npos) n += e.second;
    return n;
}
void fake_reset() { g_launches.clear(); }

static dim3_ s_grid, s_block;
static size_t s_lds;
static void *s_stream;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void *s) {
    s_grid = g, s_block = b, s_lds = lds, s_stream = s;
    return 0;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *lds, void **s) {
    *g = s_grid, *b = s_block, *lds = s_lds, *s = s_stream;
    return 0;
}
void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    g_names[host] = name;
}
int hipLaunchKernel(const void *f, dim3_, dim3_, void **, size_t, void *) {
    ++g_launches[g_names[f]];
    return 0;
}
int hipMalloc(void **p, size_t bytes) { return take(p, bytes); }
int hipHostMalloc(void **p, size_t bytes, unsigned) { return take(p, bytes); }
int hipFree(void *p) { return give(p); }
int hipHostFree(void *p) { return give(p); }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { std::memcpy(d, s, n); return 0; }
int hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)1 << 40; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(void **, const void *) { return 1; }
int hipEventCreate(void **e) { return take(e, 1); }
int hipEventCreateWithFlags(void **e, unsigned) { return take(e, 1); }
int hipEventDestroy(void *e) { return give(e); }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.0f; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **, unsigned) { return 1; }
int hipStreamDestroy(void *) { return 1; }
int hipStreamBeginCapture(void *, int) { return 1; }
int hipStreamEndCapture(void *, void **) { return 1; }
int hipGraphInstantiate(void **, void *, void *, char *, size_t) { return 1; }
int hipGraphLaunch(void *, void *) { return 1; }
int hipGraphDestroy(void *) { return 1; }
int hipGraphExecDestroy(void *) { return 1; }
}
