// A stand-in for the HIP runtime on the CPU, loaded ahead of the library so
// that its host code (streams, events, staging, launch shapes) can be tested
// without a GPU.  Device memory is host memory.  A stream is a queue whose
// work runs only when something waits for it, so that whatever the host code
// fails to order happens in the worst order.  Of the kernels, those that move
// data between host and device or count steps are modelled; the others only
// leave a line in the log.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "impl.hpp"

using namespace edp;

namespace {
std::recursive_mutex mu;
struct Stream;
struct Op {
  std::function<void()> run;
  int64_t id;
};
struct Stream {
  int n, dev;
  std::deque<Op> q;
};
struct Event {
  Stream* s = nullptr;
  int64_t id = 0;
};
std::map<int, Stream> null_streams;  // the legacy default stream of each device
std::vector<Stream*> streams;
std::map<const void*, std::string> kernels;
std::map<char*, size_t> pinned;
std::string lines;
int64_t next_id = 1;
int n_cu = 8;
thread_local int device = 0;
thread_local hipError_t last = hipSuccess;
// the launch (or copy) to fail, and the one to call back at
std::string fail_name, hook_name;
int fail_nth = 0, hook_nth = 0;
void (*hook)() = nullptr;

Stream* stream_of(hipStream_t s) {
  if (s) return (Stream*)s;
  Stream& d = null_streams[device];
  d.n = 0;
  d.dev = device;
  return &d;
}
void drain(Stream* s, int64_t upto) {
  while (!s->q.empty() && s->q.front().id <= upto) {
    Op op = s->q.front();
    s->q.pop_front();
    op.run();
  }
}
int64_t push(Stream* s, std::function<void()> f) {
  s->q.push_back({std::move(f), next_id});
  return next_id++;
}
void say(const char* fmt, ...) {
  char t[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(t, sizeof t, fmt, ap);
  va_end(ap);
  lines += t;
}
bool is_pinned(const void* p) {
  for (auto& r : pinned)
    if ((char*)p >= r.first && (char*)p < r.first + r.second) return true;
  return false;
}
// true: this call is to fail
bool event_at(const std::string& name) {
  if (hook && name.find(hook_name) != std::string::npos && --hook_nth == 0) {
    auto f = hook;
    hook = nullptr;
    mu.unlock();  // the callback may run other threads
    f();
    mu.lock();
  }
  return !fail_name.empty() && name.find(fail_name) != std::string::npos && --fail_nth == 0;
}

void gather(const GatherParts& P, int n) {
  for (int k = 0; k < n; ++k)
    if (P.p[k].sel == 0) memcpy(P.p[k].dst, P.p[k].src, (size_t)P.p[k].n * 8);
}
void small_volt(const BlockRole* r, int n) {
  for (int b = 0; b < n; ++b)
    for (int i = 0; i < r[b].j; ++i) {
      const int64_t at = (r[b].c->step + i) % kVoltChunk;
      const_cast<double*>(r[b].c->volt)[at] = r[b].c->volt_host[at];
    }
}

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
};
thread_local std::vector<Config> configs;
}  // namespace

extern "C" {

// ---- the tests' side ------------------------------------------------------
void model_cus(int n) { n_cu = n; }
const char* model_log() { return lines.c_str(); }
void model_clear() { lines.clear(); }
void model_fail(const char* name, int nth) { fail_name = name, fail_nth = nth; }
void model_hook(const char* name, int nth, void (*f)()) { hook_name = name, hook_nth = nth, hook = f; }
int model_device() { return device; }
const double* model_volt(const CaseDev* c) { return c->volt; }  // the device's V(t_s)
int64_t model_step(const CaseDev* c) { return c->step; }
void model_arrays(const CaseDev* c, int sp, void** out) {
  const SpeciesDev& S = c->sp[sp];
  void* a[6] = {S.x[0], S.vx[0], S.vy[0], S.vz[0], S.uid[0], S.vp2[0]};
  memcpy(out, a, sizeof a);
}
void model_finish() {
  std::lock_guard<std::recursive_mutex> l(mu);
  for (Stream* s : streams) drain(s, INT64_MAX);
  for (auto& d : null_streams) drain(&d.second, INT64_MAX);
}

// ---- launches ---------------------------------------------------------------
void** __hipRegisterFatBinary(const void*) { return (void**)calloc(1, 8); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  configs.push_back({g, b, lds, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = configs.back().grid, *b = configs.back().block, *lds = configs.back().lds, *st = configs.back().st;
  configs.pop_back();
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const std::string name = kernels[f];
  if (event_at(name)) return last = hipErrorLaunchFailure;
  Stream* s = stream_of(st);
  say("launch %s dev=%d stream=%d grid=%d block=%d\n", name.c_str(), device, s->n, (int)g.x, (int)b.x);
  if (device != s->dev) return last = hipErrorInvalidResourceHandle;
  std::function<void()> run = [] {};
  if (name.find("k_gather") != std::string::npos) {
    const GatherParts P = *(const GatherParts*)a[1];
    const int n = (int)g.x;
    run = [P, n] { gather(P, n); };
  } else if (name.find("k_small_volt") != std::string::npos) {
    const BlockRole* r = *(const BlockRole**)a[0];
    const int n = (int)g.x;
    run = [r, n] { small_volt(r, n); };
  } else if (name.find("k_small_end") == std::string::npos && name.find("k_small") != std::string::npos) {
    const BlockRole* r = *(const BlockRole**)a[0];
    const int n = (int)g.x;
    run = [r, n] {
      for (int k = 0; k < n; ++k) r[k].c->step += r[k].j;
    };
  } else if (name.find("k_window_end") != std::string::npos) {
    const BlockRole* r = *(const BlockRole**)a[0];
    const int n = (int)g.x, steps = *(const int*)a[1];
    run = [r, n, steps] {
      for (int k = 0; k < n; ++k) r[k].c->step += steps;
    };
  } else if (name.find("k_zero") != std::string::npos) {
    int64_t* p = *(int64_t**)a[0];
    const int64_t n = *(const int64_t*)a[1];
    run = [p, n] { memset(p, 0, (size_t)n * 8); };
  }
  push(s, run);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t lds, hipStream_t st, hipEvent_t, hipEvent_t,
                              int) {
  return hipLaunchKernel(f, g, b, a, lds, st);
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "modelled error"; }
// Static LDS of the particle kernels (of the others: not asked for).
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void* f) {
  const std::string& name = kernels[f];
  const bool electrons = name.find("k_particlesILi0") != std::string::npos, wide = name.find("ELi512E") != std::string::npos;
  memset(a, 0, sizeof *a);
  a->sharedSizeBytes = electrons ? (wide ? 23624 : 12360) : (wide ? 9288 : 5192);
  return hipSuccess;
}
// As the runtime counts: by 1024 particle threads and 160 KiB of LDS a CU, to the byte.
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t lds) {
  hipFuncAttributes a;
  (void)hipFuncGetAttributes(&a, f);
  *n = std::min<int>(1024 / b, (int)(163840 / (lds + a.sharedSizeBytes)));
  say("occupancy\n");
  return hipSuccess;
}

// ---- devices and memory -----------------------------------------------------
hipError_t hipGetDeviceCount(int* n) { return *n = 2, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = device, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = n_cu;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096), hipSuccess; }
hipError_t hipFree(void* p) {
  model_finish();
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  (void)hipMalloc(p, n);
  pinned[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  pinned.erase((char*)p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* m = calloc(16384, 64);
  return *p = m, hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::lock_guard<std::recursive_mutex> l(mu);
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (event_at(is_pinned(s) ? "copy from pinned" : "copy")) return hipErrorInvalidValue;
  if (is_pinned(s)) say("upload stream=%d\n", stream_of(st)->n);
  if (is_pinned(s) || is_pinned(d)) {
    push(stream_of(st), [=] { memcpy(d, s, n); });
  } else {  // pageable memory is read by the call
    auto t = std::make_shared<std::vector<char>>((const char*)s, (const char*)s + n);
    push(stream_of(st), [=] { memcpy(d, t->data(), n); });
  }
  return hipSuccess;
}

// ---- streams and events -------------------------------------------------------
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  streams.push_back(new Stream{(int)streams.size() + 1, device, {}});
  *s = (hipStream_t)streams.back();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  Stream* s = stream_of(st);
  say("wait stream=%d dev=%d\n", s->n, s->dev);
  drain(s, INT64_MAX);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const Event v = *(Event*)e;
  if (v.s) push(stream_of(st), [v] { drain(v.s, v.id); });
  say("order stream=%d\n", stream_of(st)->n);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t) new Event, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  Event* v = (Event*)e;
  v->s = stream_of(st);
  v->id = push(v->s, [] {});
  say("record stream=%d\n", v->s->n);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const Event* v = (Event*)e;
  return v->s && !v->s->q.empty() && v->s->q.front().id <= v->id ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const Event v = *(Event*)e;
  if (v.s) drain(v.s, v.id);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { return *t = 0.0f, hipSuccess; }

// ---- graphs: not modelled -----------------------------------------------------
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}
