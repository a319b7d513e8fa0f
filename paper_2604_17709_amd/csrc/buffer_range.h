// Offsets of the weight loads that go through a buffer descriptor: a scalar byte offset for the k position
// and a 32-bit offset per lane.  Plain C++: the host tests compile this header by itself.
#pragma once

#if defined(__HIPCC__)
#define DEINFER_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DEINFER_HOST_DEVICE inline
#endif

namespace deinfer {

// Lane offset of a load that is to read zeros: not below the size of any descriptor of the T <= 128 kernels, whose
// host code refuses factors and activations of 2^31 bytes and more (sizes are multiples of 16).  The T > 128 kernel
// does not use what its dead weight loads bring.
constexpr unsigned BUF_DEAD = 0x7ffffff0u;

struct BufOffsets { unsigned lane, scalar; };

// The load of packed weights at byte `scalar` of the k range.  live: the k-block is one of the product's (the
// same in every lane).  A load that is not live must read zeros.  The range check compares the lane offset with
// the descriptor's size LESS the scalar offset, and a scalar offset beyond the size would make that difference
// wrap: a dead load therefore takes the scalar offset 0.
DEINFER_HOST_DEVICE BufOffsets weight_load(bool live, unsigned lane, unsigned scalar) {
  return BufOffsets{lane | (live ? 0u : BUF_DEAD), live ? scalar : 0u};      // (two scalar selects and one vector instruction)
}

}  // namespace deinfer
