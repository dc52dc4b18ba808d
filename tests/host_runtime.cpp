// A stand-in for the GPU runtime in tests of the library's host code, for a
// process without a GPU: memory is host memory, launches do nothing and are
// counted, and the words that a build reads back are given by the test.
// Loaded with global visibility before libfmm.so, whose calls it then takes.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

namespace {
thread_local bool no_memory = false;
int device = 0, launches = 0;
std::string calls;
std::vector<std::vector<uint32_t>> counts;  // one set per event wait
size_t next_counts = 0;
unsigned char *pinned = nullptr;
void note(const char *what, int v) { calls += what + std::to_string(v) + " "; }
void *memory(size_t n) { return calloc(1, n ? n : 1); }
}  // namespace

void *operator new(size_t n) {
    void *p = no_memory ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}

extern "C" {
// the test's side
void rt_counts(const uint32_t *w, int n) { counts.emplace_back(w, w + n); }
void rt_forget_counts() { counts.clear(), next_counts = 0; }
int rt_launches() { return launches; }
const char *rt_calls() { return calls.c_str(); }
void rt_no_memory(int on) { no_memory = on != 0; }

// the library's side (0 is success)
int hipGetDevice(int *d) { *d = device; return 0; }
int hipSetDevice(int d) { note("set", device = d); return 0; }
int hipDeviceSynchronize() { note("wait", device); return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipDeviceGetDefaultMemPool(void **p, int) { *p = &device; return 0; }
int hipMemPoolSetAttribute(void *, int, void *) { return 0; }
const char *hipGetErrorString(int) { return "error"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { static void *s = memory(64u << 20); *p = s; return 0; }
int hipMalloc(void **p, size_t n) { *p = memory(n); return 0; }
int hipMallocAsync(void **p, size_t n, void *) { *p = memory(n); return 0; }
int hipFreeAsync(void *p, void *) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = pinned = (unsigned char *)memory(n); return 0; }
int hipHostFree(void *) { note("unpin", 0); return 0; }
int hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return 0; }
int hipMemcpy(void *, const void *, size_t, int) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = memory(1); return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = memory(1); return 0; }
int hipGraphInstantiate(void **e, void *, void **, char *, size_t) { *e = memory(1); return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphLaunch(void *, void *) { ++launches; return 0; }
int hipEventCreate(void **e) { *e = memory(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = memory(1); return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
int hipEventSynchronize(void *) {
    if (pinned && next_counts < counts.size()) {
        memcpy(pinned, counts[next_counts].data(), 4 * counts[next_counts].size());
        ++next_counts;
    }
    return 0;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
struct Dim { uint32_t x, y, z; };
static thread_local Dim g_grid, g_block;
int __hipPushCallConfiguration(Dim g, Dim b, size_t, void *) { g_grid = g; g_block = b; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *shm, void **st) {
    *g = g_grid;
    *b = g_block;
    *shm = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void *, Dim, Dim, void **, size_t, void *) { ++launches; return 0; }
}
