// A stand-in for the HIP runtime on a machine without a GPU: device memory is
// host memory, kernels are only recorded, and errors behave as HIP's do (a
// failed call leaves its error until hipGetLastError takes it; a call that
// succeeds does not clear it).  Loaded before libdfr.so, its symbols are the
// ones the library binds to.
#include <dlfcn.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

// The library's own estimate of a tile's LDS (a symbol it exports, so that this
// one takes its place): counted, then made by the library.
static int g_estimates = 0;
static void *g_library = nullptr;
namespace dfr {
struct FramePlan;
struct TileShape;
int estimate_lds_floats(const FramePlan &P, int32_t h, int32_t w, const TileShape &s, int interp) {
  using Fn = int (*)(const FramePlan &, int32_t, int32_t, const TileShape &, int);
  static const Fn real = reinterpret_cast<Fn>(
      dlsym(g_library, "_ZN3dfr19estimate_lds_floatsERKNS_9FramePlanEiiRKNS_9TileShapeEi"));
  ++g_estimates;
  return real(P, h, w, s, interp);
}
}  // namespace dfr

extern "C" {

void fake_set_library(const char *path) { g_library = dlopen(path, RTLD_LAZY | RTLD_NOLOAD); }
int fake_estimates() { return g_estimates; }

typedef int hipError_t;
struct dim3_ {
  unsigned x, y, z;
};

static int g_last = 0, g_capturing = 0, g_fail_malloc = 0, g_fail_launch = 0,
           g_skip_launches = 0;
static int g_mallocs = 0, g_host_mallocs = 0, g_copies = 0, g_graph_launches = 0;
static std::map<const void *, std::string> g_names;
static std::string g_log;  // kernels launched, one name a line

static hipError_t done(int e) {
  if (e) g_last = e;
  return e;
}

// ---- the tests' controls
void fake_reset() {
  g_last = g_capturing = g_fail_malloc = g_fail_launch = g_skip_launches = 0;
  g_mallocs = g_host_mallocs = g_copies = g_graph_launches = 0;
  g_log.clear();
}
void fake_set_capturing(int on) { g_capturing = on; }
void fake_fail_malloc(int n) { g_fail_malloc = n; }  // the next n device allocations fail
void fake_fail_launch(int n) { g_fail_launch = n; }  // the next n launches, after skipped ones
void fake_skip_launches(int n) { g_skip_launches = n; }
int fake_mallocs() { return g_mallocs; }
int fake_host_mallocs() { return g_host_mallocs; }
int fake_copies() { return g_copies; }
int fake_graph_launches() { return g_graph_launches; }
int fake_last_error() { return g_last; }
const char *fake_log() { return g_log.c_str(); }

// ---- HIP
hipError_t hipGetLastError() {
  const int e = g_last;
  g_last = 0;
  return e;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return 0;
}
hipError_t hipMalloc(void **p, size_t n) {
  ++g_mallocs;  // requests, granted or not
  if (g_capturing) return done(900);
  if (g_fail_malloc > 0) {
    --g_fail_malloc;
    return done(2);
  }
  *p = std::malloc(n < (256u << 20) ? n : 256u << 20);  // (only its first part is written here)
  return 0;
}
hipError_t hipFree(void *p) {
  std::free(p);
  return 0;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  ++g_host_mallocs;
  if (g_capturing) return done(900);
  *p = std::malloc(n);
  return 0;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return 0;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, int, void *) {
  ++g_copies;
  if (!g_capturing) std::memcpy(dst, src, n);
  return 0;
}
hipError_t hipStreamIsCapturing(void *, int *status) {
  *status = g_capturing;
  return 0;
}
hipError_t hipStreamSynchronize(void *) { return g_capturing ? done(900) : 0; }
hipError_t hipEventCreate(void **e) {
  *e = std::malloc(1);
  return 0;
}
hipError_t hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(void *e) {
  std::free(e);
  return 0;
}
hipError_t hipEventRecord(void *, void *) { return 0; }
hipError_t hipEventSynchronize(void *) { return g_capturing ? done(907) : 0; }
hipError_t hipEventElapsedTime(float *ms, void *, void *) {
  *ms = 1.0f;
  return 0;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static char scratch[8 << 20];
  *p = scratch;
  return 0;
}
hipError_t hipLaunchKernel(const void *f, dim3_ grid, dim3_ block, void **, size_t, void *) {
  if (grid.x * (uint64_t)block.x > 0xffffffffull) return done(9);  // the limit of a launch
  if (g_skip_launches > 0) {
    --g_skip_launches;
  } else if (g_fail_launch > 0) {
    --g_fail_launch;
    return done(9);
  }
  g_log += g_names[f] + "\n";
  return 0;
}
hipError_t hipGraphCreate(void **g, unsigned) {
  *g = std::malloc(1);
  return 0;
}
hipError_t hipGraphDestroy(void *g) {
  std::free(g);
  return 0;
}
hipError_t hipGraphAddKernelNode(void **node, void *, const void *, size_t, const void *) {
  *node = nullptr;
  return 0;
}
hipError_t hipGraphInstantiate(void **exec, void *, void *, char *, size_t) {
  *exec = std::malloc(1);
  return 0;
}
hipError_t hipGraphExecDestroy(void *e) {
  std::free(e);
  return 0;
}
// (a launch into a capturing stream runs at once, it is not recorded)
hipError_t hipGraphLaunch(void *, void *) {
  ++g_graph_launches;
  return 0;
}

// ---- what the compiler's host code calls
static struct {
  dim3_ grid, block;
  size_t lds;
  void *stream;
} g_config;
hipError_t __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void *stream) {
  g_config = {grid, block, lds, stream};
  return 0;
}
hipError_t __hipPopCallConfiguration(dim3_ *grid, dim3_ *block, size_t *lds, void **stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *stream = g_config.stream;
  return 0;
}
void **__hipRegisterFatBinary(const void *) {
  static void *module;
  return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}

}  // extern "C"
