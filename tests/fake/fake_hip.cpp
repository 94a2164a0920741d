// A HIP runtime in host memory, for tests of the library's host side on a
// machine without a GPU: allocations come from the heap (with a limit, so
// that they can fail), copies are made at once, and every launch, wait and
// allocation is logged by stream.  Kernels do not run; the few whose results
// the host needs to go on are stood in for: an enumeration finds every
// configuration valid (every n-th with fake_every(n)), the check of a model's inputs is made, and a draw
// publishes configuration 0 (unless fake_publish(0)).
//
// The entry points stand in front of the real runtime's when this library is
// loaded with RTLD_GLOBAL before libcgs.so.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <unordered_map>

#include "internal.h"

namespace {

std::string g_log;
std::unordered_map<const void *, std::string> g_kernel; // host function -> mangled name
std::unordered_map<void *, size_t> g_live;
std::unordered_map<const void *, int> g_lds;            // attribute of a kernel
std::map<std::string, int> g_stream;                    // address -> number
size_t g_used = 0, g_limit = (size_t)1 << 46;
bool g_publish = true;
size_t g_host_limit = SIZE_MAX;
uint32_t g_every = 1;
dim3 g_grid, g_block;
size_t g_shared;
hipStream_t g_on;

void note(const char *what, hipStream_t s, const std::string &more = "") {
  char at[32];
  snprintf(at, sizeof at, "%p", (void *)s);
  const int n = g_stream.emplace(at, (int)g_stream.size()).first->second;
  g_log += std::string(what) + " " + std::to_string(n) + (more.empty() ? "" : " " + more) + "\n";
}

hipError_t take(void **p, size_t n, size_t limit) {
  if (g_used + n > limit) return hipErrorOutOfMemory;
  *p = std::calloc(1, n ? n : 1); // pages come with their first use
  g_used += n;
  g_live[*p] = n;
  return hipSuccess;
}
hipError_t give(void *p) {
  auto it = g_live.find(p);
  if (it == g_live.end()) return hipErrorInvalidValue;
  g_used -= it->second;
  g_live.erase(it);
  std::free(p);
  return hipSuccess;
}

template <typename T> T arg(void **args, int i) { return *static_cast<T *>(args[i]); }

void publish(cgs::DrawResult *r, uint64_t seq) {
  if (!g_publish) return;
  const uint64_t part[4] = {0, 0, 1, 0}; // configuration 0 of a total weight of 1
  for (int i = 0; i < 4; ++i) r->word[i] = part[i] << 32 | (uint32_t)seq;
}

void run(const std::string &k, void **args) {
  auto is = [&](const char *name) { return k.find(name) != std::string::npos; };
  if (is("enum_mark")) {
    const auto *sp = arg<const cgs::SpaceDev *>(args, 0);
    auto *mask = arg<uint32_t *>(args, 6);
    auto *count = arg<uint32_t *>(args, 7);
    for (uint32_t t = 0; t < arg<uint32_t>(args, 5); ++t) count[t] = 0;
    if (g_every > 1) std::memset(mask, 0, sp->n_words * 4);
    for (uint64_t i = 0; i < sp->n_raw; i += g_every == 1 ? 32 : g_every) {
      const uint64_t n = g_every > 1 ? 1 : sp->n_raw - i >= 32 ? 32 : sp->n_raw - i;
      mask[i / 32] |= (n == 32 ? ~0u : (1u << n) - 1u) << (g_every > 1 ? i % 32 : 0);
      count[i / cgs::kEnumTile] += (uint32_t)n;
    }
  } else if (is("9enum_scan")) {
    const auto *count = arg<const uint32_t *>(args, 0);
    auto *off = arg<uint32_t *>(args, 2);
    uint64_t sum = 0;
    for (uint32_t t = 0; t < arg<uint32_t>(args, 1); ++t) {
      off[t] = (uint32_t)sum;
      sum += count[t];
    }
    *arg<uint64_t *>(args, 3) = sum;
  } else if (is("12enum_compact") && g_every > 1) {
    const auto *sp = arg<const cgs::SpaceDev *>(args, 0);
    auto *idx = arg<uint32_t *>(args, 3);
    for (uint64_t i = 0; i < sp->n_raw; i += g_every) *idx++ = (uint32_t)i;
  } else if (is("11check_begin")) {
    *arg<uint64_t *>(args, 0) = ~0ull;
  } else if (is("12check_floats")) {
    const auto *x = arg<const float *>(args, 0);
    auto *first = arg<uint64_t *>(args, 3);
    for (uint64_t i = 0; i < arg<uint64_t>(args, 1) && *first == ~0ull; ++i)
      if (!std::isfinite(x[i]) || (arg<int>(args, 2) && !(x[i] >= 0.0f))) *first = i;
  } else if (is("11draw_scores")) {
    publish(arg<cgs::DrawResult *>(args, 14), arg<uint64_t>(args, 15));
  } else if (is("10draw_array")) {
    publish(arg<cgs::DrawResult *>(args, 6), arg<uint64_t>(args, 7));
  } else if (is("10small_step")) {
    const auto &a = *static_cast<const cgs::SmallStep *>(args[0]);
    for (int i = 0; i < a.series.n; ++i) publish(a.res + i, a.seq0 + i);
  } else if (is("10batch_draw")) {
    const auto *d = arg<const cgs::BatchSess *>(args, 0);
    const auto *st = arg<const cgs::BatchStep *>(args, 1);
    for (uint32_t i = 0; i < g_grid.x; ++i) publish(d[i].res, st[i].seq);
  } else if (is("11batch_small")) {
    const auto *jobs = arg<const cgs::SmallJob *>(args, 1);
    auto *res = arg<cgs::DrawResult *>(args, 3);
    for (uint32_t i = 0; i < g_grid.x / arg<uint32_t>(args, 2); ++i)
      for (int k = 0; k < jobs[i].n_draws; ++k) publish(res + i * cgs::kMaxDrawSeries + k, jobs[i].seq0 + k);
  } else if (is("10batch_tune")) { // every run ends at once
    for (uint32_t i = 0; i < g_grid.x; ++i)
      static_cast<const cgs::TuneArgs *>(args[1])->run[i].state = cgs::kTuneEnded;
  } else if (is("7nb_step")) {
    const auto &a = *static_cast<const cgs::NbFused *>(args[0]);
    if (a.draw) publish(a.res, a.seq);
  }
}

} // namespace

// the library's own (it binds to these before the C++ runtime's)
void *operator new(size_t n) {
  if (n > g_host_limit) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

const char *fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }
void fake_limit(size_t bytes_left) { g_limit = g_used + bytes_left; }
size_t fake_used() { return g_used; }
void fake_host_limit(size_t bytes) { g_host_limit = bytes; } // larger host allocations fail
void fake_publish(int on) { g_publish = on != 0; }
void fake_every(unsigned n) { g_every = n; }

void **__hipRegisterFatBinary(const void *) {
  static void *h;
  return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, uint3 *, uint3 *,
                           dim3 *, dim3 *, int *) {
  g_kernel[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  g_grid = g, g_block = b, g_shared = s, g_on = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
  *g = g_grid, *b = g_block, *s = g_shared, *st = g_on;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t lds, hipStream_t s) {
  g_grid = grid;
  const std::string &k = g_kernel[f];
  note("launch", s, k);
  auto it = g_lds.find(f); // a launch may not exceed what the kernel was last allowed
  if (it != g_lds.end() && lds > (size_t)it->second) return hipErrorInvalidValue;
  run(k, args);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
  g_lds[f] = v;
  note("attr", nullptr, g_kernel[f] + " " + std::to_string(v));
  return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) {
  const hipError_t e = take(p, n, g_limit);
  note("malloc", nullptr, std::to_string(n) + (e == hipSuccess ? "" : " refused"));
  return e;
}
hipError_t hipFree(void *p) {
  note("free", nullptr);
  return give(p);
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  note("pin", nullptr, std::to_string(n));
  return take(p, n, SIZE_MAX); // the limit is the device's
}
hipError_t hipHostFree(void *p) { return give(p); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  note("copy", st);
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
  note("set", st);
  std::memset(d, v, n);
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  note("end", s);
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  note("wait", s);
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) {
  note("launch", s, "graph");
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

hipError_t hipEventCreate(hipEvent_t *e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static void *block = std::calloc(1, (size_t)1 << 25);
  *p = block;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) {
  return e == hipErrorOutOfMemory ? "out of memory" : e == hipSuccess ? "no error" : "error";
}

} // extern "C"
