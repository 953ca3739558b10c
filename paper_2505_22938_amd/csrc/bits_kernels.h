// Kernels of the bit-plane path (bitplane.h) for one key type: the plain
// form, one workgroup per tile of one image.  Included by one source per key
// type, which instantiates every variant for it.
#pragma once

#include <hip/hip_runtime.h>

#include "bitplane.h"
#include "mf_internal.h"

namespace mf {

// Second launch bound: waves per SIMD.  The largest variants need all of
// the 256 registers that two waves leave each other.
template <int KT, int G, int P>
__global__ __launch_bounds__(BitsGeo<G>::NT, P > 24 ? 2 : P > 12 ? 3 : 4) void mf_bits_kernel(ImageDesc a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bits_body<KT, G, P>(a, xcd_tile(blockIdx.x, gridDim.x), smem);
}

template <int KT>
PlainKernelFn pick_bits_variant(int v) {
  switch (v) {
#define MF_BITS_CASE(I, G, P) \
  case I: return mf_bits_kernel<KT, G, P>;
    MF_BITS_VARIANTS(MF_BITS_CASE)
#undef MF_BITS_CASE
    default: return nullptr;
  }
}

}  // namespace mf
