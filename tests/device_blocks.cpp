// Calls of the library on a stand-in for the HIP runtime: allocations from host
// memory with a switch that makes them fail, copies that are copies, launches that do
// nothing. The definitions here come before the runtime library's, so liblqcd.so
// uses them. Exit status 0: the case named on the command line holds.
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../include/lqcd.h"

static std::map<void*, size_t> live;  // device blocks handed out
static size_t live_bytes = 0;
static long frees = 0;
static bool full = false;       // no memory until a block is freed
static long fail_at = -1;       // the allocation of this number (from now) fails
static bool no_heap = false;    // operator new throws
static bool copying = false;    // a copy from the caller's memory may still run

void* operator new(size_t n) {
  void* p = no_heap ? nullptr : std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

struct Dim3 {
  uint32_t x, y, z;
};

extern "C" {
int hipMalloc(void** p, size_t n) {
  if (full || (fail_at >= 0 && fail_at-- == 0)) return 2;
  const bool heap = no_heap;
  no_heap = false;
  *p = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  live[*p] = n ? n : 1;
  no_heap = heap;
  live_bytes += n;
  return 0;
}
int hipFree(void* p) {
  if (!p) return 0;
  auto it = live.find(p);
  if (it == live.end()) std::abort();  // not a block of ours, or freed before
  live_bytes -= it->second;
  munmap(p, it->second);
  live.erase(it);
  ++frees;
  full = false;
  copying = false;
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? 0 : 2; }
int hipHostFree(void* p) { return std::free(p), 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) {
  if (n <= (size_t)1 << 24) std::memcpy(d, s, n);
  if (kind == 1) copying = true;
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void*) {
  if (n <= (size_t)1 << 24) std::memset(p, v, n);
  return 0;
}
int hipStreamSynchronize(void*) { return copying = false, 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "stand-in"; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipGetSymbolAddress(void** p, const void*) {
  static char scratch[256];
  return *p = scratch, 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return *s = (void*)1, 0; }
int hipStreamDestroy(void*) { return 0; }
int hipEventCreate(void** e) { return *e = (void*)1, 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return *e = (void*)1, 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) { return *t = 1.f, 0; }
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*) { return 0; }
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
  return *g = *b = Dim3{1, 1, 1}, *s = 0, *st = nullptr, 0;
}
}

#define OK(call)                                                                               \
  do {                                                                                         \
    const int s_ = (call);                                                                     \
    if (s_ != LQCD_OK) {                                                                       \
      no_heap = false;                                                                         \
      std::printf("%s: status %d (%s)\n", #call, s_, lqcd_last_error());                       \
      std::exit(1);                                                                            \
    }                                                                                          \
  } while (0)

static lqcd_ctx* context(int lx, int ly, int lz, int lt) {
  const int dims[4] = {lx, ly, lz, lt};
  lqcd_ctx* c = nullptr;
  OK(lqcd_create(dims, -1, nullptr, &c));
  double* dev = nullptr;  // launches do nothing: the links are never read
  OK(lqcd_set_gauge(c, reinterpret_cast<double*>(&dev), 1));
  OK(lqcd_set_clover(c, 0.1, 0.0));
  return c;
}

static const lqcd_dwf_params DWF = [] {
  lqcd_dwf_params d{};
  d.Ls = 4;
  d.M5 = 1.8;
  d.mf = 0.05;
  d.b5 = 1.5;
  d.c5 = 0.5;
  return d;
}();

// A call that needs no heap memory to succeed neither throws nor ends the program for want of it
static int no_heap_case() {
  lqcd_ctx* c = context(4, 4, 4, 4);
  std::vector<double> a(256 * 24 * 4), b(a);
  for (int k = 0; k < 3; ++k) {
    no_heap = true;
    OK(lqcd_stag_apply(c, LQCD_STAG_D, k & 1, 0.1, a.data(), b.data(), 0));
    OK(lqcd_dwf_apply(c, &DWF, 0, k & 1, a.data(), b.data(), 0));
    no_heap = false;
  }
  lqcd_destroy(c);
  return live.empty() ? 0 : 1;
}

// A call that fails for want of memory has no copy from the caller's memory under way
static int failed_copy_case() {
  std::vector<double> a(256 * 24 * 4), b(a);
  for (int call = 0; call < 6; ++call)
    for (int n = 0, failed = 1; failed; ++n) {
      lqcd_ctx* c = context(4, 4, 4, 4);
      fail_at = n;
      int s = LQCD_OK;
      switch (call) {
        case 0: s = lqcd_dwf_apply(c, &DWF, 0, 0, a.data(), b.data(), 0); break;
        case 1: s = lqcd_dwf_apply_schur(c, &DWF, 0, 0, a.data(), b.data(), 0); break;
        case 2: s = lqcd_dwf_solve(c, &DWF, a.data(), b.data(), nullptr, nullptr); break;
        case 3: s = lqcd_dwf_solve_eo(c, &DWF, a.data(), b.data(), nullptr, nullptr); break;
        case 4: s = lqcd_stag_apply(c, LQCD_STAG_D, 0, 0.1, a.data(), b.data(), 0); break;
        case 5: s = lqcd_stag_solve(c, 0.1, a.data(), b.data(), nullptr, nullptr); break;
      }
      failed = fail_at < 0;  // the allocation of that number was asked for
      fail_at = -1;
      if (failed && s != LQCD_ENOMEM) return std::printf("call %d, allocation %d: status %d\n", call, n, s), 1;
      if (copying) return std::printf("call %d, allocation %d: a copy is under way\n", call, n), 1;
      lqcd_destroy(c);
    }
  return live.empty() ? 0 : 1;
}

// Where memory has run out, idle blocks of any context are given back, whichever call asks
static int reclaim_case() {
  std::vector<double> a(256 * 24 * 4), b(a);
  lqcd_sap_params sap{};
  sap.block[0] = 4, sap.block[1] = sap.block[2] = sap.block[3] = 4;
  sap.ncycles = sap.nmr = 1;
  const double* bs = a.data();
  double* xs = b.data();
  const int one = 1;
  double gbs = 0;
  lqcd_ctx* other = nullptr;
  const int dims[4] = {4, 4, 4, 4};
  for (int call = 0; call < 7; ++call)
    for (int mine = 0; mine < 2; ++mine) {
      lqcd_ctx *c = context(8, 8, 8, 8), *d = context(4, 4, 4, 4);
      std::vector<double> f(4096 * 24), g(f);
      bs = f.data(), xs = g.data();
      OK(lqcd_stag_apply(mine ? c : d, LQCD_STAG_D, 0, 0.1, f.data(), g.data(), 0));
      full = true;
      switch (call) {
        case 0: OK(lqcd_apply_native(c, LQCD_DPREC_SCHUR, 2, f.data(), g.data())); break;
        case 1: OK(lqcd_solve(c, f.data(), g.data(), nullptr, nullptr)); break;
        case 2: OK(lqcd_apply_sap(c, &sap, f.data(), g.data(), 0)); break;
        case 3: OK(lqcd_solve_batch(&c, &one, &bs, &xs, 1, nullptr, nullptr)); break;
        case 4: OK(lqcd_bandwidth_probe(c, 1, 1 << 20, 1, &gbs)); break;
        case 5: OK(lqcd_create(dims, -1, nullptr, &other)); lqcd_destroy(other); break;
        case 6: {
          std::vector<double> h(4096 * 24 * 4), k(h);
          OK(lqcd_dwf_apply_schur(c, &DWF, 0, 1, h.data(), k.data(), 0));
        }
      }
      if (full) return std::printf("call %d asked for no memory\n", call), 1;
      lqcd_destroy(c);
      lqcd_destroy(d);
      if (!live.empty()) return std::printf("call %d: blocks left\n", call), 1;
    }
  return 0;
}

// A context's idle blocks stay within 2 GiB and those of all contexts within 16 GiB, the
// ones idle longest go first, and a context's go with it
static int bound_case() {
  double* dev = nullptr;
  double* any = reinterpret_cast<double*>(&dev);
  lqcd_dwf_params d = DWF;
  constexpr int N = 12;
  lqcd_ctx* c[N];
  size_t last = 0;  // bytes of the last context without idle blocks
  for (int k = 0; k < N; ++k) {
    last = live_bytes;
    c[k] = k % 3 ? context(32, 32, 32, 32) : context(16, 32, 32, 32);
    last = live_bytes - last;
  }
  const size_t base = live_bytes;
  size_t most = 0;
  for (int k = 0; k < 4 * N; ++k) {
    d.Ls = 1 + (k / N + k) % 4;
    OK(lqcd_dwf_apply(c[k % N], &d, 0, k & 1, any, any + 1, 1));
    if (live_bytes - base > (size_t)16 << 30) return std::printf("%zu bytes idle\n", live_bytes - base), 1;
    most = live_bytes - base > most ? live_bytes - base : most;
  }
  if (most <= (size_t)12 << 30) return std::printf("%zu bytes kept at most\n", most), 1;
  for (int k = 0; k < N - 1; ++k) lqcd_destroy(c[k]);
  for (int k = 0; k < 8; ++k) {  // one context alone
    d.Ls = 1 + k % 4;
    OK(lqcd_dwf_apply(c[N - 1], &d, 0, k & 1, any, any + 1, 1));
    if (live_bytes - last > (size_t)2 << 30) return std::printf("%zu bytes of one context\n", live_bytes - last), 1;
  }
  const long before = frees;
  OK(lqcd_dwf_apply(c[N - 1], &d, 0, 1, any, any + 1, 1));  // the last call again: its blocks are there
  if (frees != before) return std::printf("a kept block was freed\n"), 1;
  lqcd_destroy(c[N - 1]);
  return live.empty() ? 0 : 1;
}

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "no_heap") return no_heap_case();
  if (name == "failed_copy") return failed_copy_case();
  if (name == "reclaim") return reclaim_case();
  if (name == "bound") return bound_case();
  return 2;
}
