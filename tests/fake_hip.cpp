// A HIP runtime without a GPU, for tests of the host code: device memory is host memory, kernels are recorded and not
// run, and the few kernels that answer the host through pinned memory answer here.  Failures are planted by count.
// Linked with the library's own objects into one shared object whose references bind inside it.
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "ae_internal.h"
#include "dense_tile.h"

namespace {

struct Launch {
  std::string name;
  unsigned gx, gy, threads;
};

std::map<const void *, std::string> g_names;
std::vector<Launch> g_launches;
std::map<void *, size_t> g_live;
int g_device = 0, g_malloc_device = -1;   // current one, that of the last device allocation
hipError_t g_last = hipSuccess;
long g_fail_launch = -1;     // launches until one fails
size_t g_fail_alloc = 0;     // device allocations of this size and more fail (0: none)
size_t g_room = 0;           // device memory that there is (0: no end of it)
bool g_go_on = true;         // answer of the exit rule
bool g_mute = false;         // no kernel answers
bool g_capture = false;      // streams are being captured: launches are recorded for later, waiting is an error
int g_syncs = 0;             // stream synchronisations
struct { dim3 grid, block; size_t shm; hipStream_t s; } g_call;

hipError_t note(hipError_t e) {
  if (e != hipSuccess) g_last = e;   // an error stays until it is read
  return e;
}

bool is(const std::string &name, const char *kernel) { return name.find(kernel) != std::string::npos; }

template <typename T>
T arg(void **args, int i) { return *reinterpret_cast<T *>(args[i]); }

}  // namespace

extern "C" {

// ---- what a test asks
int fake_launches() { return (int)g_launches.size(); }
const char *fake_name(int i) { return g_launches[i].name.c_str(); }
void fake_grid(int i, unsigned *gx, unsigned *gy, unsigned *threads) {
  *gx = g_launches[i].gx; *gy = g_launches[i].gy; *threads = g_launches[i].threads;
}
void fake_clear() { g_launches.clear(); }
void fake_fail_launch(long after) { g_fail_launch = after; }
void fake_fail_alloc(size_t bytes) { g_fail_alloc = bytes; }
void fake_room(size_t bytes) { g_room = bytes; }
void fake_set_error(int e) { g_last = (hipError_t)e; }
int fake_last_error() { return (int)g_last; }
void fake_mute(int mute) { g_mute = mute != 0; }
void fake_capture(int on) { g_capture = on != 0; }
int fake_syncs() { return g_syncs; }
void fake_set_device(int d) { g_device = d; }
int fake_device() { return g_device; }
int fake_malloc_device() { return g_malloc_device; }
void fake_rule(int go_on) { g_go_on = go_on != 0; }
size_t fake_live_bytes() {
  size_t t = 0;
  for (auto &a : g_live) t += a.second;
  return t;
}

// ---- device code that host code can follow
int fake_dense_slot(int w, int i, int nw, int dm) { return ae::dense_slot(w, i, nw, dm); }
int fake_dense_source(int slot, int rb0, int RB) { return ae::dense_source(slot, rb0, RB); }

// ---- registration and launches
void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
  g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shm, hipStream_t s) {
  g_call.grid = grid; g_call.block = block; g_call.shm = shm; g_call.s = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shm, hipStream_t *s) {
  *grid = g_call.grid; *block = g_call.block; *shm = g_call.shm; *s = g_call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
  if (g_fail_launch >= 0 && g_fail_launch-- == 0) return note(hipErrorLaunchOutOfResources);
  const std::string &name = g_names[f];
  g_launches.push_back(Launch{name, grid.x, grid.y, block.x});
  if (g_mute || g_capture) return hipSuccess;
  if (is(name, "export_row_kernel")) {
    memcpy(arg<float *>(args, 2), arg<const float *>(args, 0), arg<size_t>(args, 1) * sizeof(float));
    for (unsigned p = 0; p < grid.x; ++p) arg<uint32_t *>(args, 3)[p] = arg<uint32_t>(args, 4);
  } else if (is(name, "publish_state_kernel")) {
    auto *m = arg<ae::HostMirror *>(args, 1);
    m->st = *arg<const ae::DevState *>(args, 0);
    m->published = arg<uint32_t>(args, 2);
  } else if (is(name, "ldlp_tail_kernel")) {
    auto *m = arg<ae::HostMirror *>(args, 10);
    m->st = *arg<const ae::DevState *>(args, 9);
    m->published = arg<uint32_t>(args, 11);
  } else if (is(name, "set_state_kernel")) {
    memcpy(arg<float *>(args, 2), arg<const float *>(args, 0), arg<int>(args, 1) * sizeof(float));
    arg<ae::HostMirror *>(args, 6)->imported = arg<uint32_t>(args, 7);
  } else if (is(name, "argmax_finish_kernel")) {
    const auto d = arg<ae::DddFinish>(args, 7);
    if (d.flag) *d.flag = d.seq << 1 | (g_go_on ? 1u : 0u);
  }
  return hipSuccess;
}

// ---- memory
hipError_t hipMalloc(void **p, size_t n) {
  if ((g_fail_alloc && n >= g_fail_alloc) || (g_room && fake_live_bytes() + n > g_room)) return note(hipErrorOutOfMemory);
  *p = calloc(1, n);
  g_live[*p] = n;
  g_malloc_device = g_device;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  g_live.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static std::vector<float> stage((size_t)AE_KV_IMPORT_STATIC_MAX_FLOATS);
  *p = stage.data();
  return hipSuccess;
}

// ---- the rest
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipPeekAtLastError() { return g_last; }
const char *hipGetErrorString(hipError_t) { return "planted"; }
hipError_t hipGetDevice(int *d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  ++g_syncs;
  return g_capture ? note(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)calloc(1, 8); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }

}  // extern "C"
