// slab_copy.hpp -- one launch that copies several result slabs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace eat {

struct SlabCopy {
  const int32_t *src;  // 16-byte aligned
  int32_t *dst;        // memory of the current device
  int32_t words;
};
constexpr int kCopySlabs = 64;
struct CopyList {
  int32_t n;
  SlabCopy e[kCopySlabs];
};
static_assert(sizeof(CopyList) <= 2048, "the list travels in the kernel arguments");

hipError_t launch_copy_slabs(const CopyList &l, hipStream_t stream);

}  // namespace eat
