// A client of libozfp4.so with a stand-in for the HIP runtime (its
// definitions, in the executable, come before the runtime library's), for
// tests/test_launch_errors_host.py. Launches are queued and take effect at the
// next wait, as on a stream; only the line maxima have one: they set the flag
// word they were given if the call was armed as non-finite. One launch can be
// made to fail. Every entry point with a flag word is run with each of its
// launches failing; the call after it has to succeed.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "ozfp4.h"

typedef int hipError_t;
typedef void* hipStream_t;
struct Dim3 { unsigned x, y, z; };

// kernels by their host address; the library registers them before this
// file's own objects are constructed
static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}
static std::vector<int*> g_queue;    // flag words of the queued line maxima, armed calls only
static bool g_armed = false;         // the call's inputs hold a NaN
static int g_launches = 0, g_fail_at = 0, g_device_waits = 0;
static hipError_t g_last = 0;

static void drain() {
  for (int* flag : g_queue) *flag = 1;
  g_queue.clear();
}

extern "C" {
hipError_t __hipPushCallConfiguration(Dim3, Dim3, size_t, hipStream_t) { return 0; }
hipError_t __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, hipStream_t* st) {
  *g = Dim3{1, 1, 1}; *b = Dim3{1, 1, 1}; *s = 0; *st = nullptr;
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, hipStream_t) {
  if (++g_launches == g_fail_at) return g_last = 1;
  if (g_armed && names()[f].find("k_line_max") != std::string::npos)
    g_queue.push_back(*static_cast<int**>(args[4]));
  return 0;
}
hipError_t hipGetLastError(void) { hipError_t e = g_last; g_last = 0; return e; }
hipError_t hipStreamSynchronize(hipStream_t) { drain(); return 0; }
hipError_t hipDeviceSynchronize(void) { ++g_device_waits; drain(); return 0; }
hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
hipError_t hipEventCreate(void** e) { *e = nullptr; return 0; }
hipError_t hipEventDestroy(void*) { return 0; }
hipError_t hipEventElapsedTime(float* t, void*, void*) { *t = 0; return 0; }
hipError_t hipEventRecord(void*, hipStream_t) { return 0; }
hipError_t hipEventSynchronize(void*) { return 0; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return 0; }
hipError_t hipFree(void* p) { std::free(p); return 0; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return 0; }
hipError_t hipHostFree(void* p) { std::free(p); return 0; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = std::malloc(OZFP4_SCRATCH_BYTES);
  return 0;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return 0; }
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, hipStream_t) {
  return 0;
}
hipError_t hipGetDevice(int* d) { *d = 0; return 0; }
hipError_t hipSetDevice(int) { return 0; }
hipError_t hipStreamIsCapturing(hipStream_t, int* s) { *s = 0; return 0; }
}

static char g_buf[64];   // operands and results: no kernel runs

static int run(int entry) {
  const int64_t m = 300, n = 200, k = 500;
  double* d = reinterpret_cast<double*>(g_buf);
  float* f = reinterpret_cast<float*>(g_buf);
  uint8_t* u = reinterpret_cast<uint8_t*>(g_buf);
  int32_t* i = reinterpret_cast<int32_t*>(g_buf);
  switch (entry) {
    case 0: return ozfp4_dgemm(m, n, k, d, m, d, k, d, m, 18);
    case 1: return ozfp4_dgemm_noalloc(m, n, k, d, m, d, k, d, m, 18);
    case 2: return ozfp4_dgemm_split(m, n, k, d, m, d, k, d, m, 19);
    case 3: return ozfp4_dgemm_ozi(m, n, k, d, m, d, k, d, m, 15);
    case 4: return ozfp4_sgemm(m, n, k, f, m, f, k, f, m, 10);
    case 5: return ozfp4_scales(m, n, k, d, m, d, k, 18, i, i);
    case 6: return ozfp4_limb_planes(m, n, k, d, m, d, k, 18, u, u);
    case 7: return ozfp4_residues(m, n, k, d, m, d, k, 18, u, m);
    case 8: return ozfp4_ozi_limb_planes(m, n, k, d, m, d, k, 15, u, u);
    default: return ozfp4_ozi_partials(m, n, k, d, m, d, k, 15, reinterpret_cast<int64_t*>(g_buf), m);
  }
}
constexpr int kEntries = 10;

static int call(int entry, bool armed, int fail_at) {
  g_armed = armed;
  g_launches = 0;
  g_fail_at = fail_at;
  const int rc = run(entry);
  g_armed = false;
  g_fail_at = 0;
  return rc;
}

#define CHECK(c, e, x)                                                          \
  do {                                                                          \
    if (!(c)) {                                                                 \
      std::printf("entry %d, launch %d: %s (%d)\n", e, fail, #c, x);            \
      return 1;                                                                 \
    }                                                                           \
  } while (0)

int main() {
  int fail = 0, rc;
  if ((rc = ozfp4_init()) != OZFP4_OK) { std::printf("init %d\n", rc); return 1; }
  int failures = 0;
  for (int e = 0; e < kEntries; ++e) {
    fail = 0;
    g_device_waits = 0;
    rc = call(e, false, 0);
    CHECK(rc == OZFP4_OK, e, rc);
    const int launches = g_launches;
    rc = call(e, true, 0);
    CHECK(rc == OZFP4_ENONFINITE, e, rc);
    rc = call(e, false, 0);
    CHECK(rc == OZFP4_OK, e, rc);
    if (e == 0) g_device_waits = 0;               // the workspace may have grown
    CHECK(e != 0 || (call(e, false, 0) == OZFP4_OK && g_device_waits == 0), e, g_device_waits);
    for (fail = 1; fail <= launches; ++fail) {
      rc = call(e, true, fail);                   // ends early, line maxima still queued
      CHECK(rc == OZFP4_EHIP, e, rc);
      ++failures;
      rc = call(0, false, 0);
      CHECK(rc == OZFP4_OK, e, rc);
    }
  }
  std::printf("%d\n", failures);
  return 0;
}
