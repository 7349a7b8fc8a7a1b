// slab_copy.hip -- copies of finished result slabs to the callers' device
// buffers, many slabs in one launch.
#include "slab_copy.hpp"

namespace eat {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

// Bound by the launch, not by the copy: a serving step's slabs are some tens of
// 40-200 KB copies, each less than a microsecond of HBM time but 5 us of host
// time as a copy of its own.  One list of them travels in the kernel arguments;
// work-group (x, y) copies the x-th kCopyWords words of slab y, 16 bytes a lane
// where the destination allows it.
constexpr int kCopyWords = 256 * 4 * 4;

__global__ __launch_bounds__(256) void k_copy_slabs(CopyList l) {
  const SlabCopy c = l.e[blockIdx.y];
  const int32_t base = (int32_t)blockIdx.x * kCopyWords;
  if (base >= c.words) return;
  const int32_t n = min(c.words - base, kCopyWords);
  const int32_t *src = c.src + base;  // 256-byte aligned slots
  int32_t *dst = c.dst + base;
  int32_t done = 0;
  if ((reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
    const int32_t n4 = n >> 2;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t i = (int32_t)threadIdx.x + 256 * k;
      if (i < n4) reinterpret_cast<v4i *>(dst)[i] = reinterpret_cast<const v4i *>(src)[i];
    }
    done = n4 << 2;
  }
  for (int32_t i = done + (int32_t)threadIdx.x; i < n; i += 256) dst[i] = src[i];
}

}  // namespace

hipError_t launch_copy_slabs(const CopyList &l, hipStream_t stream) {
  if (l.n <= 0) return hipSuccess;
  if (l.n > kCopySlabs) return hipErrorInvalidValue;
  int32_t words = 0;
  for (int32_t i = 0; i < l.n; ++i) words = words < l.e[i].words ? l.e[i].words : words;
  if (words <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)(((int64_t)words + kCopyWords - 1) / kCopyWords);
  hipLaunchKernelGGL(k_copy_slabs, dim3(blocks, (unsigned)l.n), dim3(256), 0, stream, l);
  return hipGetLastError();
}

}  // namespace eat
