// journeys.hip -- the query variants of Section I beside the single-source
// answer: the journey (earliest arrival path) behind every arrival time, and
// the profile of a source over an interval of departure times.  Both run the
// relaxation's own lookup device functions (next departure of a connection
// type at or after a time, Sections II-B..II-D).
#include "relax.hpp"

namespace eat {
namespace {

// ---------------------------------------------------------------------------
// Parents.  The arrival arr[v] (v != s) of an EAT answer is realised by a
// connection (u, v, t, lam) with arr[u] <= t and t + lam == arr[v].  Within a
// connection type (u, v, lam) the only candidate is its first departure at or
// after arr[u]: a later one arrives later.  The parent is the realising one with
// the smallest (u, lam).
//
// The answer array is its own scratch: par[3v ..] starts as -1 three times, a
// first pass over the reached stops' types takes the unsigned minimum of u on
// par[3v], a second one, over the types whose tail won, that of lam on par[3v + 2]
// and the maximum of t = arr[v] - lam on par[3v + 1].
//
// What bounds it is latency: a few hundred to a few thousand of the stops are
// reached, each with some fifteen types of three dependent reads.  A wave takes
// 16 stops and spreads the types of the reached ones over its lanes, 16 lanes a
// stop, so that no lane has more than a few in a row (one thread per stop walked
// all of a stop's types, 12 us on city-50k; the two passes take 4.4 each).
// ---------------------------------------------------------------------------
constexpr int kParentStops = 16;  // stops of a wave

template <int KIND, bool LAM>
__global__ __launch_bounds__(256) void k_parents(GraphDev Gd, const int32_t *arr, int32_t s, int32_t *par) {
  __shared__ int4 todo[256 / 64][kParentStops];  // {u, arr[u], first type, type count}
  const GraphG G = graph_g(Gd);
  gp<const int32_t> A = (gp<const int32_t>)arr;
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  const int64_t u64 = ((int64_t)blockIdx.x * (256 / 64) + wave) * kParentStops + lane;
  const bool mine = lane < kParentStops && u64 < G.n_vertices;
  const int32_t u = mine ? (int32_t)u64 : 0;
  const int32_t x = mine ? A[u] : INF;
  const uint64_t m = __ballot(x != INF);
  if (m == 0) return;
  if (x != INF) {
    const int2 r = G.vt[u];
    todo[wave][__popcll(m & ((1ull << lane) - 1ull))] = make_int4(u, x, r.x, r.y);
  }
  __builtin_amdgcn_wave_barrier();  // one wave's LDS operations stay in order
  const int32_t n = (int32_t)__popcll(m);
  for (int32_t i = lane >> 4; i < n; i += 4) {
    const int4 e = todo[wave][i];
    for (int32_t j = e.z + (lane & 15); j < e.z + e.w; j += 16) {
      int4 rec;
      if constexpr (KIND == kKindGrid) rec = G.side[j];  // {v, lam, ..}
      else rec = G.ty[2 * (int64_t)j];                   // {v, lam, ..}
      const int32_t v = rec.x, lam = rec.y;
      if (v == s) continue;
      const int32_t av = A[v];
      if (av == INF || (int64_t)e.y + lam > av) continue;  // no departure at or after arr[u] can realise av
      if constexpr (LAM) {
        if (par[3 * (int64_t)v] != e.x) continue;  // a smaller tail realises it
      }
      Ctr c;
      const int32_t tc = next_departure<KIND>(G, j, e.z, e.w, e.y, c);
      if (tc == INF || (int64_t)tc + lam != av) continue;
      if constexpr (LAM) {
        atomicMax(par + 3 * (int64_t)v + 1, tc);
        atomicMin(reinterpret_cast<unsigned int *>(par + 3 * (int64_t)v + 2), (unsigned int)lam);
      } else {
        atomicMin(reinterpret_cast<unsigned int *>(par + 3 * (int64_t)v), (unsigned int)e.x);
      }
    }
  }
}

// p[0 .. n) = x; the 16-byte stores cover what lies between 16-byte boundaries.
__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t x) {
  const int64_t head = min(n, (int64_t)(((16 - (reinterpret_cast<uintptr_t>(p) & 15u)) & 15u) >> 2));
  const int64_t n4 = (n - head) >> 2, tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  gp<v4i> p4 = (gp<v4i>)(p + head);
  const v4i x4 = {x, x, x, x};
  for (int64_t i = tid; i < n4; i += (int64_t)gridDim.x * blockDim.x) p4[i] = x4;
  if (tid < head) p[tid] = x;
  const int64_t tail = head + 4 * n4 + tid;
  if (tid < 4 && tail < n) p[tail] = x;
}

// ---------------------------------------------------------------------------
// Profiles.  The distinct departures of s in [lo, hi], in increasing order, by
// one work-group: every thread walks the departures of its connection types in
// chunks of kDepSpan seconds and sets a bit per departure in LDS; the bits'
// prefix sum gives each departure its place.  out[0..cap) receives the first cap
// of them; info[0] = their count, info[1] = the first departure after hi (INF if
// none); out and info are host memory (a graph's scratch) or device memory.
//
// What bounds it is the longest chain of one type's departures, one read each (a
// wave that took the minimum over the types for every departure in turn made 32
// steps of 0.7 us for 32 departures, this takes 4.6 us; the types' own chains are a few long).
// ---------------------------------------------------------------------------
constexpr int32_t kDepSpan = 1 << 17;  // seconds of a chunk: a day and a half
constexpr int kDepBlock = 256;

template <int KIND>
__global__ __launch_bounds__(kDepBlock) void k_departures(GraphDev Gd, int32_t s, int32_t lo, int32_t hi, int32_t cap,
                                                          int32_t *out, int32_t *info) {
  constexpr int kWords = kDepSpan / 32;
  __shared__ uint32_t bits[kWords];
  __shared__ int32_t wsum[kDepBlock / 64], next;
  const GraphG G = graph_g(Gd);
  const int2 r = G.vt[s];
  const int tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
  int32_t from = lo, found = 0;
  for (;;) {
    // the chunk [from, to]
    const int32_t to = (int64_t)from + kDepSpan - 1 < hi ? from + kDepSpan - 1 : hi;
    const int words = ((to - from) >> 5) + 1, per = (words + kDepBlock - 1) / kDepBlock;  // per: of a thread, consecutive
    for (int i = tid; i < words; i += kDepBlock) bits[i] = 0u;
    if (tid == 0) next = INF;
    __syncthreads();
    for (int32_t j = r.x + tid; j < r.x + r.y; j += kDepBlock) {
      int32_t x = from;
      for (;;) {
        Ctr c;
        const int32_t t = next_departure<KIND>(G, j, r.x, r.y, x, c);
        if (t == INF || t > to) {
          atomicMin(&next, t);
          break;
        }
        atomicOr(&bits[(uint32_t)(t - from) >> 5], 1u << ((uint32_t)(t - from) & 31u));
        x = t + 1;  // t < INF
      }
    }
    __syncthreads();
    const int32_t after = next;
    int32_t mine = 0;
    const int w0 = min(tid * per, words), w1 = min(w0 + per, words);
    for (int i = w0; i < w1; ++i) mine += __popc(bits[i]);
    const int32_t incl = wave_incl_sum(mine);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int32_t place = found + incl - mine;
    for (int w = 0; w < kDepBlock / 64; ++w) {
      if (w < wave) place += wsum[w];
      found += wsum[w];
    }
    if (mine) {
      for (int i = w0; i < w1; ++i) {
        uint32_t b = bits[i];
        while (b) {
          if (place < cap) out[place] = from + i * 32 + (__ffs(b) - 1);
          ++place;
          b &= b - 1u;
        }
      }
    }
    if (after == INF || after > hi) {
      if (tid == 0) {
        info[0] = found;
        info[1] = after;
      }
      return;
    }
    from = after;  // the next departure starts the next chunk
    __syncthreads();
  }
}

// Row i of the k x V profile matrix keeps arr[i][v] only where it beats row
// i + 1 (the last row: the query at the first departure after the interval,
// `later`, or nothing when there is none); each thread walks one column, eight
// rows' reads in flight at a time (one at a time the walk was a chain of k read
// latencies: 17 us for 32 rows of city-50k, now 6.5).
__global__ __launch_bounds__(256) void k_profile_filter(int32_t *arr, const int32_t *later, int32_t k, int32_t V, int32_t s) {
  constexpr int kRows = 8;
  for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < V; v += gridDim.x * blockDim.x) {
    int32_t a = arr[v];
    for (int32_t i0 = 0; i0 < k; i0 += kRows) {
      int32_t b[kRows];  // rows i0 + 1 .. i0 + kRows
#pragma unroll
      for (int i = 0; i < kRows; ++i) {
        const int32_t row = i0 + 1 + i;
        b[i] = row < k ? arr[(int64_t)row * V + v] : (row == k && later ? later[v] : INF);
      }
#pragma unroll
      for (int i = 0; i < kRows; ++i) {
        if (i0 + i < k) {
          arr[(int64_t)(i0 + i) * V + v] = (v != s && a < b[i]) ? a : INF;
          a = b[i];
        }
      }
    }
  }
}

int blocks_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

}  // namespace

template <int KIND>
static void launch_parents_kind(const GraphDev &g, const int32_t *arr, int32_t s, int32_t *par, hipStream_t stream) {
  const unsigned blocks = (unsigned)(((int64_t)g.n_vertices + 4 * kParentStops - 1) / (4 * kParentStops));
  hipLaunchKernelGGL((k_parents<KIND, false>), dim3(blocks), dim3(256), 0, stream, g, arr, s, par);
  hipLaunchKernelGGL((k_parents<KIND, true>), dim3(blocks), dim3(256), 0, stream, g, arr, s, par);
}

hipError_t launch_parents(const GraphDev &g, int kind, const int32_t *arr, int32_t s, int32_t *par,
                          hipStream_t stream) {
  const int32_t V = g.n_vertices;
  if (V <= 0) return hipSuccess;
  if (kind != kKindGrid && kind != kKindCompact && kind != kKindFlat) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for((3 * (int64_t)V + 3) / 4)), dim3(256), 0, stream, par, 3 * (int64_t)V, -1);
  if (kind == kKindGrid) launch_parents_kind<kKindGrid>(g, arr, s, par, stream);
  else if (kind == kKindCompact) launch_parents_kind<kKindCompact>(g, arr, s, par, stream);
  else launch_parents_kind<kKindFlat>(g, arr, s, par, stream);
  return hipGetLastError();
}

hipError_t launch_departures(const GraphDev &g, int kind, int32_t s, int32_t lo, int32_t hi, int32_t cap,
                             int32_t *out, int32_t *info, hipStream_t stream) {
  if (kind == kKindGrid)
    hipLaunchKernelGGL(k_departures<kKindGrid>, dim3(1), dim3(kDepBlock), 0, stream, g, s, lo, hi, cap, out, info);
  else if (kind == kKindCompact)
    hipLaunchKernelGGL(k_departures<kKindCompact>, dim3(1), dim3(kDepBlock), 0, stream, g, s, lo, hi, cap, out, info);
  else if (kind == kKindFlat)
    hipLaunchKernelGGL(k_departures<kKindFlat>, dim3(1), dim3(kDepBlock), 0, stream, g, s, lo, hi, cap, out, info);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_profile_filter(int32_t *arr, const int32_t *later, int32_t k, int32_t V, int32_t s,
                                 hipStream_t stream) {
  if (k <= 0 || V <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_profile_filter, dim3(blocks_for(V)), dim3(256), 0, stream, arr, later, k, V, s);
  return hipGetLastError();
}

}  // namespace eat
