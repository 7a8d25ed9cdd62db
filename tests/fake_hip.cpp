// A HIP runtime for tests of the library's host code without a GPU: device memory is host
// memory, copies are copies, kernels do nothing, streams, events and graphs are empty. Built
// as a shared library and loaded (RTLD_GLOBAL) before libstarred.so, whose undefined HIP
// symbols then resolve to these. It counts the live allocations, can fail the n-th one to
// come, and keeps the sources of device-to-device copies and the names of the kernels launched.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::map<void *, size_t> live;
long long live_bytes = 0, fail_in = -1, mallocs = 0;
int last_error = 0;
std::vector<const void *> copy_src;
std::map<const void *, std::string> kernels;
std::string launches;
struct Dim3 { uint32_t x, y, z; };
struct { Dim3 grid, block; size_t shmem; void *stream; } call;
}  // namespace

extern "C" {
// ---- what a test reads and sets ----
long long fake_live_count() { return (long long)live.size(); }
long long fake_live_bytes() { return live_bytes; }
long long fake_mallocs() { return mallocs; }
void fake_fail_malloc_in(long long n) { fail_in = n; }  // the n-th from now (1: the next); < 0: none
long long fake_copies_from(const void *src)
{
    long long n = 0;
    for (const void *s : copy_src) n += s == src;
    return n;
}
const char *fake_launches()  // since the last call: mangled names, a space after each
{
    static std::string out;
    out.swap(launches);
    launches.clear();
    return out.c_str();
}

// ---- memory ----
int hipMalloc(void **p, size_t n)
{
    ++mallocs;
    if (fail_in > 0 && --fail_in == 0) {
        fail_in = -1;
        *p = nullptr;
        return last_error = 2;  // hipErrorOutOfMemory
    }
    *p = calloc(1, n ? n : 1);
    live[*p] = n;
    live_bytes += (long long)n;
    return 0;
}
int hipFree(void *p)
{
    if (!p) return 0;
    auto it = live.find(p);
    if (it == live.end()) abort();  // freed twice, or never allocated
    live_bytes -= (long long)it->second;
    live.erase(it);
    free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *)
{
    if (kind == 3) copy_src.push_back(s);  // hipMemcpyDeviceToDevice
    memcpy(d, s, n);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *)
{
    static char symbol[4 << 20];
    *p = symbol;
    return 0;
}

// ---- kernels ----
void *__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void *, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    kernels[f] = name;
}
void __hipRegisterVar(void *, void *, char *, const char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void *) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void *st) { call = {g, b, s, st}; return 0; }
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *s, void **st)
{
    *g = call.grid;
    *b = call.block;
    *s = call.shmem;
    *st = call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **, size_t, void *)
{
    launches += kernels[f] + " ";
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return 0; }

// ---- device, streams, events, graphs ----
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }  // (only compute units are asked for)
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int) { return "fake error"; }
int hipStreamCreate(void **s) { *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.f; return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(void **x, void *, void *, char *, size_t) { *x = malloc(1); return 0; }
int hipGraphUpload(void *, void *) { return 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *g) { free(g); return 0; }
int hipGraphExecDestroy(void *x) { free(x); return 0; }
}
