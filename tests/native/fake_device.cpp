// A host stand-in for the device under session.cpp: the HIP calls that it makes
// and the library functions that it uses, on host memory.  A query's answer is
// one number in every word of its slab, written when it is launched.  Work on
// the streams of callers can be held back (events recorded there stay pending),
// and any of its calls can be made to fail, from the test.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "device.hpp"
#include "eat.h"
#include "internal.hpp"
#include "slab_copy.hpp"

namespace {

std::map<std::string, long> ctl;  // settings and counters, by name
std::string error_text;
std::set<const void *> own_streams;  // the session's: their work is done at once
std::map<const char *, size_t> device_memory;
struct Event {
  int pending = 0;
};
struct Op {
  std::function<void()> run;
};
std::deque<Op> held;

bool fails(const char *what) { return ctl[what] > 0 && --ctl[what] == 0; }
void drain() {
  while (!held.empty()) {
    held.front().run();
    held.pop_front();
  }
}
void enqueue(const void *stream, std::function<void()> f) {
  if (ctl["hold"] && !own_streams.count(stream)) held.push_back(Op{std::move(f)});
  else f();
}
int32_t answer(int32_t graph, int32_t s, int32_t ts) { return 1000000 * graph + 1000 * s + ts; }

}  // namespace

extern "C" {

void fake_set(const char *name, long v) { ctl[name] = v; }
long fake_get(const char *name) { return ctl[name]; }
void fake_drain() { drain(); }
const char *fake_error() { return error_text.c_str(); }
int32_t *fake_alloc(size_t words) {
  void *p = nullptr;
  (void)hipMalloc(&p, words * 4);
  return static_cast<int32_t *>(p);
}
eat_graph *fake_graph(int32_t n_vertices) {
  eat_graph *g = new eat_graph();
  g->info.n_vertices = g->desc.n_vertices = n_vertices;
  return g;
}

hipError_t hipMalloc(void **p, size_t n) {
  *p = std::malloc(n + 16);
  device_memory[static_cast<const char *>(*p)] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  device_memory.erase(static_cast<const char *>(p));
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
  *p = std::malloc(n + 16);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned int) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemset(void *p, int x, size_t n) {
  std::memset(p, x, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (!own_streams.count(st)) ++ctl["memcpys"];
  enqueue(st, [=] { std::memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  drain();
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  own_streams.insert(*s);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  own_streams.erase(s);
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  ++ctl["stream_syncs"];
  drain();
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) {
  *d = (int)ctl["stream_device"];
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event());
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event *>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  if (!own_streams.count(st) && fails("fail_record")) return hipErrorUnknown;
  Event *ev = reinterpret_cast<Event *>(e);
  ++ev->pending;
  enqueue(st, [ev] { --ev->pending; });
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  return reinterpret_cast<Event *>(e)->pending ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (reinterpret_cast<Event *>(e)->pending) drain();
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  ++ctl["attributes"];
  std::this_thread::sleep_for(std::chrono::microseconds(ctl["attributes_us"]));
  auto it = device_memory.upper_bound(static_cast<const char *>(p));
  if (it == device_memory.begin()) return hipErrorInvalidValue;
  --it;
  if (static_cast<const char *>(p) >= it->first + it->second) return hipErrorInvalidValue;
  a->type = hipMemoryTypeDevice;
  a->device = 0;
  return hipSuccess;
}

}  // extern "C"

namespace eat {

eat_status set_err(eat_status s, const std::string &m) {
  error_text = m;
  return s;
}
eat_status hip_err(hipError_t, const char *what) { return set_err(EAT_ERR_DEVICE, what); }
eat_status device_limits(int, DeviceLimits *out) {
  out->cus = 256;
  out->lds = 160 << 10;
  return EAT_OK;
}
eat_status make_plan(const eat_run_options *, int32_t, int, Plan *) { return EAT_OK; }
eat_status exec_kind(const eat_graph *const *, int32_t, int, int *kind) {
  *kind = 0;
  return EAT_OK;
}
int relax_blocks_per_cu(int, int, int, int, size_t, bool) { return 1; }
void apply_plan(const Plan &, RunArgs *) {}
int order_bands(int, int32_t, int64_t) { return -1; }
void order_queries(const std::vector<const eat_graph *> &, std::vector<QueryDev> &qs, int, std::vector<int32_t> &off, int) {
  off = {0, (int32_t)qs.size()};
}
hipError_t launch_relax(const RunArgs &a, int, int, int, int, int, size_t, hipStream_t) {
  if (fails("fail_relax")) return hipErrorUnknown;
  // "finish": only so many queries of a launch end
  for (int32_t i = 0; i < a.nq && (ctl["finish"] == 0 || i < ctl["finish"]); ++i) {
    const QueryDev &q = a.queries[i];
    for (int32_t v = 0; v < a.graphs[q.graph].n_vertices; ++v) q.arr[v] = answer(q.graph, q.s, q.ts);
    a.done[q.index] = a.epoch;
  }
  return hipSuccess;
}
hipError_t launch_copy_slabs(const CopyList &l, hipStream_t stream) {
  if (l.n <= 0) return hipSuccess;
  ++ctl["copy_launches"];
  if (fails("fail_copies")) return hipErrorUnknown;
  for (int32_t i = 0; i < l.n; ++i)  // one launch writes them all at once
    for (int32_t j = 0; j < i; ++j)
      if (l.e[i].dst < l.e[j].dst + l.e[j].words && l.e[j].dst < l.e[i].dst + l.e[i].words) ++ctl["overlaps"];
  enqueue(stream, [l] {
    for (int32_t i = 0; i < l.n; ++i) std::memcpy(l.e[i].dst, l.e[i].src, (size_t)l.e[i].words * 4);
  });
  return hipSuccess;
}

}  // namespace eat
