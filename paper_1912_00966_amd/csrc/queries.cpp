// queries.cpp -- C ABI of the query variants beside the single-source answer
// (Section I): parent connections (journeys) and profiles of a source over an
// interval of departure times.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>
#include <string>
#include <vector>

#include "device.hpp"
#include "eat.h"
#include "internal.hpp"

using eat::hip_err;
using eat::set_err;

namespace eat {
hipError_t launch_parents(const GraphDev &g, int kind, const int32_t *arr, int32_t s, int32_t *par,
                          hipStream_t stream);
hipError_t launch_departures(const GraphDev &g, int kind, int32_t s, int32_t lo, int32_t hi, int32_t cap,
                             int32_t *out, int32_t *info, hipStream_t stream);
hipError_t launch_profile_filter(int32_t *arr, const int32_t *later, int32_t k, int32_t V, int32_t s,
                                 hipStream_t stream);
}  // namespace eat

static eat_status check_graph(const eat_graph *g) {
  if (!g) return set_err(EAT_ERR_INVALID_ARGUMENT, "graph is NULL");
  int cur = -1;
  HIP_TRY(hipGetDevice(&cur));
  if (cur != g->device) return set_err(EAT_ERR_INVALID_ARGUMENT, "graph lives on another device than the current one");
  return EAT_OK;
}

extern "C" eat_status eat_parents(const eat_graph *g, int32_t s, const int32_t *arr, int32_t *par, void *stream) {
  eat_status st = check_graph(g);
  if (st != EAT_OK) return st;
  if (!arr || !par) return set_err(EAT_ERR_INVALID_ARGUMENT, "arr or par is NULL");
  if (s < 0 || s >= g->info.n_vertices) return set_err(EAT_ERR_INVALID_ARGUMENT, "source out of range");
  int kind = 0;
  st = eat::exec_kind(&g, 1, EAT_HEADERS_AUTO, &kind);
  if (st != EAT_OK) return st;
  const hipError_t e = eat::launch_parents(g->desc, kind, arr, s, par, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_err(e, "parents launch");
  return EAT_OK;
}

static eat_status too_many(int32_t k, int32_t cap, const int32_t *arr) {
  if (cap == 0 && !arr) return EAT_OK;  // the count only
  return set_err(EAT_ERR_UNSUPPORTED,
                 std::to_string(k) + " departures in the interval, cap is " + std::to_string(cap));
}

// Memory of a call that has no scratch; given back when its stream has finished.
struct OwnMemory {
  char *buf = nullptr;
  hipStream_t stream;
  explicit OwnMemory(hipStream_t s) : stream(s) {}
  ~OwnMemory() {
    if (!buf) return;
    (void)hipStreamSynchronize(stream);
    (void)hipFree(buf);
  }
};

// From the graph's scratch nothing is allocated: the departures arrive in host
// memory, then one upload, the batch, the filter and one wait.  (Allocations and
// blocking copies were 0.15 ms of a 0.37 ms profile of 32 departures.)  More
// departures than the scratch takes, or a scratch that is in use: memory of the
// call's own; a batch that does not fit it: a batch object.
static eat_status profile(const eat_graph *g, int32_t s, int32_t t_lo, int32_t t_hi, int32_t cap, int32_t *dep,
                          int32_t *n_dep, int32_t *arr, hipStream_t hs, const eat_run_options *ro) {
  eat_status st = check_graph(g);
  if (st != EAT_OK) return st;
  const int32_t V = g->info.n_vertices;
  if (!n_dep) return set_err(EAT_ERR_INVALID_ARGUMENT, "n_dep is NULL");
  if (s < 0 || s >= V) return set_err(EAT_ERR_INVALID_ARGUMENT, "source out of range");
  if (t_lo < 0 || t_hi < t_lo) return set_err(EAT_ERR_INVALID_ARGUMENT, "need 0 <= t_lo <= t_hi");
  if (cap < 0 || (cap > 0 && (!dep || !arr))) return set_err(EAT_ERR_INVALID_ARGUMENT, "cap < 0, or dep/arr NULL");
  int kind = 0;
  st = eat::exec_kind(&g, 1, ro ? ro->headers : EAT_HEADERS_AUTO, &kind);
  if (st != EAT_OK) return st;
  eat::ScratchLock lock(cap <= eat::kScratchQueries ? g : nullptr);
  eat::CallScratch *const sc = lock.get();
  OwnMemory own(hs);
  // {count, next}, the departures, the row of the query after the interval
  int32_t info[2] = {0, 0};
  std::vector<int32_t> h_dep;
  int32_t *later = nullptr;
  hipError_t e;
  if (sc) {
    e = eat::launch_departures(g->desc, kind, s, t_lo, t_hi, cap, sc->out_dev + 2, sc->out_dev, hs);
    const hipError_t w = eat::wait_scratch(sc, hs);
    if (e == hipSuccess) e = w;
    if (e != hipSuccess) return hip_err(e, "profile departures");
    info[0] = sc->out[0];
    info[1] = sc->out[1];
    h_dep.assign(sc->out + 2, sc->out + 2 + std::min(info[0], cap));
    later = sc->row;
  } else {
    const size_t b_info = eat::align_up(2 * sizeof(int32_t));
    const size_t b_dep = eat::align_up((size_t)std::max(cap, 1) * sizeof(int32_t));
    const size_t b_row = eat::align_up((size_t)V * sizeof(int32_t));
    HIP_TRY(hipMalloc(reinterpret_cast<void **>(&own.buf), b_info + b_dep + b_row));
    int32_t *d_info = reinterpret_cast<int32_t *>(own.buf);
    int32_t *d_dep = reinterpret_cast<int32_t *>(own.buf + b_info);
    later = reinterpret_cast<int32_t *>(own.buf + b_info + b_dep);
    e = eat::launch_departures(g->desc, kind, s, t_lo, t_hi, cap, d_dep, d_info, hs);
    if (e == hipSuccess) e = hipMemcpyAsync(info, d_info, sizeof(info), hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e != hipSuccess) return hip_err(e, "profile departures");
    if (info[0] <= cap) {
      h_dep.resize((size_t)info[0]);
      if (info[0] > 0) e = hipMemcpy(h_dep.data(), d_dep, h_dep.size() * sizeof(int32_t), hipMemcpyDeviceToHost);
      if (e != hipSuccess) return hip_err(e, "profile departures copy");
    }
  }
  const int32_t k = info[0], next = info[1];
  *n_dep = k;
  if (k > cap) return too_many(k, cap, arr);
  if (k == 0) return EAT_OK;
  // one batch: a query per departure, and one at the first departure after t_hi
  const int32_t nq = k + (next != EAT_INF ? 1 : 0);
  std::vector<int32_t> qg((size_t)nq, 0), qs((size_t)nq, s), qt(h_dep);
  std::vector<int32_t *> rows((size_t)nq);
  for (int32_t i = 0; i < k; ++i) rows[(size_t)i] = arr + (int64_t)i * V;
  if (nq > k) {
    qt.push_back(next);
    rows[(size_t)k] = later;
  } else {
    later = nullptr;
  }
  eat::BatchPlan bp;
  st = eat::plan_batch(&g, 1, qg.data(), qs.data(), qt.data(), nullptr, nq, rows.data(), ro, &bp);
  if (st != EAT_OK) return st;
  if (sc && eat::fits_scratch(bp, 1)) {
    e = eat::launch_from_scratch(bp, &g, 1, sc, hs);
    if (e == hipSuccess) e = eat::launch_profile_filter(arr, later, k, V, s, hs);
    const hipError_t w = eat::wait_scratch(sc, hs);
    if (e == hipSuccess) e = w;
    if (e != hipSuccess) return hip_err(e, "profile batch");
    st = eat::batch_status(sc->out[0]);
    if (st != EAT_OK) return st;
  } else {
    eat_batch *b = nullptr;
    st = eat::batch_from_plan(bp, &g, 1, nullptr, &b);
    if (st != EAT_OK) return st;
    st = eat_batch_run(b, hs);
    if (st == EAT_OK) st = eat_batch_wait(b, nullptr);
    eat_batch_free(b);
    if (st != EAT_OK) return st;
    e = eat::launch_profile_filter(arr, later, k, V, s, hs);
    const hipError_t w = hipStreamSynchronize(hs);
    if (e == hipSuccess) e = w;
    if (e != hipSuccess) return hip_err(e, "profile filter");
  }
  std::copy(h_dep.begin(), h_dep.end(), dep);
  return EAT_OK;
}

extern "C" eat_status eat_profile(const eat_graph *g, int32_t s, int32_t t_lo, int32_t t_hi, int32_t cap,
                                  int32_t *dep, int32_t *n_dep, int32_t *arr, void *stream,
                                  const eat_run_options *ro) {
  try {
    return profile(g, s, t_lo, t_hi, cap, dep, n_dep, arr, static_cast<hipStream_t>(stream), ro);
  } catch (const std::bad_alloc &) {  // nothing throws across the C ABI
    return set_err(EAT_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
}
