// A HIP runtime without a device, for tests of the library's host code on the
// CPU: device memory is host memory, kernels do nothing, and every launch,
// wait, event and graph call is logged.  A call can be made to fail, streams
// belong to devices, and events may only be recorded on streams of the device
// that was current when they were made, as on real hardware.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

struct Stream {
  int dev, prio, id;
  uint32_t mask;
  bool capturing = false;
  std::vector<std::string> rec;
};
struct Event { int dev; };
struct Graph { int id; std::vector<std::string> kernels; };

std::recursive_mutex mu;
int cur_dev = 0, n_streams = 0, n_graphs = 0, live_events = 0, live_streams = 0, live_graphs = 0;
hipError_t last_error = hipSuccess;
std::string log_text;
std::map<const void *, std::string> kernel_name;
std::map<std::string, int> fail_in;  // calls until the named one fails
struct Config { dim3 grid, block; size_t shmem; hipStream_t st; };
thread_local std::vector<Config> configs;

Stream *S(hipStream_t s) { return (Stream *)s; }
std::string sid(hipStream_t s) { return s ? "s" + std::to_string(S(s)->id) : "s0"; }
int dev_of(hipStream_t s) { return s ? S(s)->dev : cur_dev; }
void note(const std::string &what) { log_text += what + "\n"; }

// whether this call of `name` is to fail
bool fails(const char *name) {
  auto it = fail_in.find(name);
  if (it == fail_in.end() || --it->second > 0) return false;
  fail_in.erase(it);
  note(std::string("failed ") + name);
  return true;
}
#define LOCK std::lock_guard<std::recursive_mutex> lock_(mu)
#define MAY_FAIL(name) if (fails(name)) return last_error = hipErrorUnknown

std::string short_name(const char *mangled) {
  std::string s(mangled);
  size_t k = s.find("k_"), t = s.find("k3_");
  if (k == std::string::npos || (t != std::string::npos && t < k)) k = t;
  return k == std::string::npos ? s : s.substr(k, s.find('I', k) - k);
}

}  // namespace

extern "C" {

// --- what the tests call ---------------------------------------------------
void stub_reset(void) { LOCK; log_text.clear(); fail_in.clear(); last_error = hipSuccess; cur_dev = 0; }
const char *stub_log(void) { LOCK; static std::string out; out = log_text; return out.c_str(); }
void stub_clear(void) { LOCK; log_text.clear(); }
void stub_fail(const char *name, int nth) { LOCK; fail_in[name] = nth; }
void stub_device(int dev) { cur_dev = dev; }
int stub_current_device(void) { return cur_dev; }
int stub_live(int what) { LOCK; return what == 0 ? live_events : what == 1 ? live_streams : live_graphs; }
void *stub_stream(int dev, int prio, uint32_t mask) { LOCK; return new Stream{dev, prio, ++n_streams, mask}; }

// --- the runtime -----------------------------------------------------------
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void **, const void *host, char *dev, const char *, unsigned, void *, void *, void *, void *,
                           int *) {
  LOCK;
  kernel_name[host] = short_name(dev);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t st) {
  configs.push_back({grid, block, shmem, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *st) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid; *block = c.block; *shmem = c.shmem; *st = c.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **, size_t, hipStream_t st) {
  LOCK;
  MAY_FAIL("hipLaunchKernel");
  if (st && S(st)->capturing) S(st)->rec.push_back(kernel_name[fn]);
  else note("launch " + kernel_name[fn] + " " + sid(st));
  return hipSuccess;
}
hipError_t hipGetLastError(void) { LOCK; const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "stub error"; }
hipError_t hipGetDevice(int *d) { *d = cur_dev; return hipSuccess; }
hipError_t hipSetDevice(int d) { cur_dev = d; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static double buf[16384]; *p = buf; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  LOCK;
  MAY_FAIL("hipHostMalloc");
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { LOCK; note("hostfree"); std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  LOCK;
  MAY_FAIL("hipMemcpyAsync");
  std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  LOCK;
  MAY_FAIL("hipStreamCreateWithFlags");
  *s = (hipStream_t) new Stream{cur_dev, 0, ++n_streams, ~0u};
  ++live_streams;
  note("newstream " + sid(*s) + " dev" + std::to_string(cur_dev));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { LOCK; --live_streams; delete S(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  LOCK;
  MAY_FAIL("hipStreamSynchronize");
  note("sync " + sid(s));
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) { *d = dev_of(s); return hipSuccess; }
hipError_t hipStreamGetPriority(hipStream_t s, int *p) { *p = s ? S(s)->prio : 0; return hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t s, uint32_t n, uint32_t *m) {
  for (uint32_t k = 0; k < n; ++k) m[k] = s ? S(s)->mask : ~0u;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
  LOCK;
  MAY_FAIL("hipStreamWaitEvent");
  note("wait " + sid(s));
  return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  LOCK;
  MAY_FAIL("hipEventCreateWithFlags");
  *e = (hipEvent_t) new Event{cur_dev};
  ++live_events;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { LOCK; --live_events; delete (Event *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  LOCK;
  MAY_FAIL("hipEventRecord");
  if (((Event *)e)->dev != dev_of(s)) return last_error = hipErrorInvalidHandle;
  note("record " + sid(s));
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { LOCK; MAY_FAIL("hipEventSynchronize"); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }

hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *out) {
  *out = s && S(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  LOCK;
  MAY_FAIL("hipStreamBeginCapture");
  if (!s || S(s)->capturing) return last_error = hipErrorIllegalState;
  S(s)->capturing = true;
  S(s)->rec.clear();
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  LOCK;
  S(s)->capturing = false;
  *g = (hipGraph_t) new Graph{0, S(s)->rec};
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  LOCK;
  MAY_FAIL("hipGraphInstantiate");
  Graph *G = new Graph{++n_graphs, ((Graph *)g)->kernels};
  ++live_graphs;
  std::string line = "instantiate g" + std::to_string(G->id);
  for (const std::string &k : G->kernels) line += " " + k;
  note(line);
  *x = (hipGraphExec_t)G;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph *)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { LOCK; --live_graphs; delete (Graph *)x; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  LOCK;
  MAY_FAIL("hipGraphLaunch");
  if (s && S(s)->capturing) return last_error = hipErrorIllegalState;
  note("graph g" + std::to_string(((Graph *)x)->id) + " n" + std::to_string(((Graph *)x)->kernels.size()) + " " + sid(s));
  return hipSuccess;
}

}  // extern "C"
