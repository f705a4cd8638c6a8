// Stand-in for the HIP runtime on the CPU, preloaded before libllr.so: device
// memory is host memory, kernels are not run, and every launch, copy, event and
// synchronisation is recorded with its stream.  One call of a chosen kind can be
// made to fail.  Allocations of the C++ heap are counted as well.
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>

namespace {

struct Rec {
    const char* op;
    const char* name;   // kernel
    void* stream;
    size_t bytes;
};
constexpr int kMax = 1 << 20;
Rec g_rec[kMax];
long g_n = 0;
long g_news = 0;
size_t g_new_max = 0;
const char* g_fail_op = "";
long g_fail_at = -1;   // calls of g_fail_op left before the one that fails
char g_scratch[1 << 20];
uintptr_t g_next = 0x1000;   // handles of streams, events and graphs
std::map<const void*, std::string>* g_names;

int note(const char* op, void* stream = nullptr, const char* name = "", size_t bytes = 0) {
    if (g_n < kMax) g_rec[g_n] = {op, name, stream, bytes};
    ++g_n;
    if (g_fail_at >= 0 && strcmp(op, g_fail_op) == 0 && g_fail_at-- == 0) return 999;
    return 0;
}

struct Dim3 { uint32_t x, y, z; };
thread_local struct { Dim3 grid, block; size_t shmem; void* stream; } g_cfg;

}  // namespace

void* operator new(size_t n) {
    ++g_news;
    if (n > g_new_max) g_new_max = n;
    void* p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {

void rec_reset() { g_n = 0; g_news = 0; g_new_max = 0; g_fail_at = -1; }
long rec_count() { return g_n < kMax ? g_n : kMax; }
const char* rec_op(long i) { return g_rec[i].op; }
const char* rec_name(long i) { return g_rec[i].name; }
void* rec_stream(long i) { return g_rec[i].stream; }
size_t rec_bytes(long i) { return g_rec[i].bytes; }
long rec_news() { return g_news; }
size_t rec_new_max() { return g_new_max; }
void rec_fail(const char* op, long at) {
    static char keep[64];
    snprintf(keep, sizeof keep, "%s", op);
    g_fail_op = keep;
    g_fail_at = at;
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    if (!g_names) g_names = new std::map<const void*, std::string>;
    (*g_names)[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shmem, void* st) { g_cfg = {g, b, shmem, st}; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shmem, void** st) {
    *g = g_cfg.grid; *b = g_cfg.block; *shmem = g_cfg.shmem; *st = g_cfg.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void* st) {
    const auto it = g_names->find(f);
    return note("launch", st, it == g_names->end() ? "?" : it->second.c_str());
}

int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return note("hipDeviceSynchronize"); }
const char* hipGetErrorString(int) { return "made to fail"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = g_scratch; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }

int hipMalloc(void** p, size_t n) { *p = calloc(n, 1); return note("hipMalloc", nullptr, "", n); }
int hipFree(void* p) { free(p); return note("hipFree"); }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return note("hipHostMalloc", nullptr, "", n); }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return note("hipMemcpy", nullptr, "", n); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* st) { memcpy(d, s, n); return note("hipMemcpyAsync", st, "", n); }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return note("hipMemset", nullptr, "", n); }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { memset(d, v, n); return note("hipMemsetAsync", st, "", n); }

static int handle(void** h) { *h = (void*)(g_next += 16); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { handle(s); return note("hipStreamCreateWithFlags", *s); }
int hipStreamDestroy(void* s) { return note("hipStreamDestroy", s); }
int hipStreamSynchronize(void* s) { return note("hipStreamSynchronize", s); }
int hipStreamWaitEvent(void* s, void*, unsigned) { return note("hipStreamWaitEvent", s); }
int hipStreamBeginCapture(void* s, int) { return note("hipStreamBeginCapture", s); }
int hipStreamEndCapture(void* s, void** g) { handle(g); return note("hipStreamEndCapture", s); }
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return handle(e); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void* s) { return note("hipEventRecord", s); }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return 0; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { return handle(x); }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipGraphLaunch(void*, void* s) { return note("hipGraphLaunch", s); }

}  // extern "C"
