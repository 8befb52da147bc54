// A stand-in for the HIP runtime with which the library's host side runs on the CPU: the device arena is host memory, copies are
// copies, kernels are not run but recorded by name, and launches can be made to fail.  Loaded with global symbols ahead of the
// library, which then finds these functions first.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

struct dim3 { unsigned x, y, z; };
struct Launch { std::string name; int first_arg; };
static std::map<const void*, std::string>& names() { static auto* n = new std::map<const void*, std::string>; return *n; }
static std::vector<Launch>& log_() { static auto* l = new std::vector<Launch>; return *l; }
static int fail_from = -1, fail_times = 0, last_error = 0;
static struct { dim3 grid, block; size_t smem; void* stream; } config;
static long news = 0;
static bool counting = false;

void* operator new(size_t n) { if (counting) ++news; void* p = malloc(n ? n : 1); if (!p) abort(); return p; }
void* operator new(size_t n, const std::nothrow_t&) noexcept { if (counting) ++news; return malloc(n ? n : 1); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
// ---- the test's side
void fake_reset() { log_().clear(); }
int fake_count() { return (int)log_().size(); }
const char* fake_name(int i) { return log_()[i].name.c_str(); }
int fake_first_arg(int i) { return log_()[i].first_arg; }               // the first int of the kernel's first argument
void fake_fail(int from, int times) { fail_from = from; fail_times = times; }
long fake_news(int on) { const long n = news; news = 0; counting = on != 0; return n; }

// ---- the library's side
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { names()[host] = device; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { config = {g, b, s, st}; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = config.grid; *b = config.block; *s = config.smem; *st = config.stream; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, void*) {
  if (fail_from >= 0 && fail_from-- == 0) {
    if (--fail_times > 0) fail_from = 0;
    return last_error = 719;
  }
  // a grid has less than 2^32 work items along each axis
  if ((unsigned long long)g.x * b.x >> 32 || (unsigned long long)g.y * b.y >> 32 || (unsigned long long)g.z * b.z >> 32) return last_error = 9;
  const bool was = counting;
  counting = false;
  int a;
  memcpy(&a, args[0], sizeof a);
  log_().push_back({names()[f], a});
  counting = was;
  return 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "injected"; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int, void*) {
  for (size_t i = 0; i < h; ++i) memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
  return 0;
}
int hipPointerGetAttributes(void*, const void*) { return 1; }
static int handle;
int hipStreamCreateWithFlags(void** s, unsigned) { *s = &handle; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { *e = &handle; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = &handle; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return 0; }
}
