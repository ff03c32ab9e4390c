// The recorded step sequences of ge_step and ge_prepare_step against a HIP
// runtime that only counts what it is asked for and fails where it is told to
// (the definitions below stand in for the library's imports; no device).
// Started by tests/test_host_runtime.py; prints "step graphs clean".
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "grainenv.h"

static long kernels, in_capture, replays, instantiated, streams;
static bool capturing, user_captures, no_stream, no_begin, no_end, no_instance;

extern "C" {
struct dim { unsigned x, y, z; };
int __hipPushCallConfiguration(dim, dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* m, void** s) {
  *g = *b = dim{1, 1, 1};
  *m = 0;
  *s = nullptr;
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* p;
  return &p;
}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int hipLaunchKernel(const void*, dim, dim, void**, size_t, void*) {
  ++(capturing ? in_capture : kernels);
  return 0;
}
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceGetAttribute(int* v, int, int) { return *v = 256, 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 8, 0; }
int hipGetSymbolAddress(void** p, const void*) { return *p = (void*)0x1000, 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { return *p = calloc(1, n), 0; }
int hipHostFree(void* p) { return free(p), 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "as told"; }
int hipStreamIsCapturing(void*, int* s) { return *s = user_captures, 0; }
int hipStreamCreateWithFlags(void** s, unsigned) {
  if (no_stream) return 1;
  ++streams;
  return *s = (void*)0x2000, 0;
}
int hipStreamDestroy(void*) { return --streams, 0; }
int hipStreamBeginCapture(void*, int) { return no_begin ? 1 : (capturing = true, 0); }
int hipStreamEndCapture(void*, void** g) {
  capturing = false;
  return no_end ? (*g = nullptr, 1) : (*g = (void*)0x3000, 0);
}
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) {
  if (no_instance) return 1;
  ++instantiated;
  return *e = (void*)0x4000, 0;
}
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return --instantiated, 0; }
int hipGraphLaunch(void*, void*) { return ++replays, 0; }
}

#define CHECK(c)                                                 \
  do {                                                           \
    if (!(c)) {                                                  \
      printf("%s:%d: %s\n", __FILE__, __LINE__, #c);              \
      exit(1);                                                   \
    }                                                            \
  } while (0)

static ge_ctx* context() {
  ge_params p{};
  for (int a = 0; a < 3; ++a) p.hi[a] = 1e-3;
  p.lambda0 = p.h = p.rc = 5e-6;
  p.a[0] = 1e-5;
  p.b[0] = 2.0;
  p.b[1] = 3.0;
  p.branching = p.box_exit = 1;
  p.cap_particles = p.cap_stopped = 1 << 16;
  p.cap_grains = 16;
  p.cap_claim_bricks = 1 << 12;
  size_t n = 0;
  ge_ctx* c = nullptr;
  CHECK(ge_workspace_size(&p, &n) == GE_OK);
  CHECK(ge_create(&p, (void*)0x100000, n, (void*)0x5000, &c) == GE_OK);
  kernels = in_capture = replays = 0;
  return c;
}

// Kernel launches of n calls of one step without recordings.
static long plain(int n) {
  ge_ctx* c = context();
  CHECK(ge_use_graphs(c, 0) == GE_OK);
  for (int k = 0; k < n; ++k) CHECK(ge_step(c, 1e-4, 1, nullptr) == GE_OK);
  const long launched = kernels;
  ge_destroy(c);
  return launched;
}

int main() {
  const int n = 100;
  const long want = plain(n);

  // A recording that fails leaves the steps to be launched, without an error
  // and without another try for the same arguments.
  bool* fails[] = {&no_stream, &no_begin, &no_end, &no_instance};
  for (bool* f : fails) {
    ge_ctx* c = context();
    *f = true;
    for (int k = 0; k < n; ++k) CHECK(ge_step(c, 1e-4, 1, nullptr) == GE_OK);
    CHECK(kernels == want && replays == 0 && in_capture < 20);
    ge_step_stats st;
    CHECK(ge_step(c, 1e-4, 1, &st) == GE_OK);
    *f = false;
    // New arguments are recorded again.
    for (int k = 0; k < n; ++k) CHECK(ge_step(c, 2e-4, 1, nullptr) == GE_OK);
    CHECK(replays > 80);
    ge_destroy(c);
    CHECK(instantiated == 0 && streams == 0);
  }

  // A prepared context records nothing in its first calls, of one step or of
  // many.
  {
    ge_ctx* c = context();
    CHECK(ge_prepare_step(c, 1e-4) == GE_OK);
    const long recorded = in_capture;
    CHECK(recorded > 0 && kernels == 0);
    for (int k = 0; k < 15; ++k) CHECK(ge_step(c, 1e-4, 1, nullptr) == GE_OK);
    CHECK(replays == 15);
    CHECK(ge_step(c, 1e-4, 1, nullptr) == GE_OK);  // the 16th step ends with a re-sort
    CHECK(replays == 15);
    CHECK(ge_step(c, 1e-4, 64, nullptr) == GE_OK);
    CHECK(replays == 19 && in_capture == recorded);
    ge_destroy(c);
    CHECK(instantiated == 0 && streams == 0);
  }

  // Steps on a stream that the caller captures are launched into it.
  {
    ge_ctx* c = context();
    user_captures = true;
    for (int k = 0; k < n; ++k) CHECK(ge_step(c, 1e-4, 1, nullptr) == GE_OK);
    user_captures = false;
    CHECK(kernels == want && replays == 0 && in_capture == 0);
    ge_destroy(c);
  }
  printf("step graphs clean\n");
  return 0;
}
