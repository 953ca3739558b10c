// Kernels of the bit-plane path (bitplane.h) for one key type: the plain
// form, one workgroup per tile of one image, and the form of batch plans, one
// workgroup per entry of a tile queue.  Each key type and form has a source
// that instantiates every variant for it.
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

// As the batched tile kernels: the descriptor is read through the constant
// address space, field by field with scalar loads.
template <int KT, int G, int P>
__global__ __launch_bounds__(BitsGeo<G>::NT, P > 24 ? 2 : P > 12 ? 3 : 4) void mf_bits_batched_kernel(
    ConstDesc* descs, const int2* __restrict__ queue, int begin, int, int*, unsigned char*, long long) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int2 q = queue[begin + blockIdx.x];
  const int img = __builtin_amdgcn_readfirstlane(q.x);
  const int tile = __builtin_amdgcn_readfirstlane(q.y);
  bits_body<KT, G, P>(descs[img], tile, smem);
}

template <int KT>
PlainKernelFn pick_bits_variant(int v) {
  switch (v) {
#define MF_BITS_CASE(I, G, P) \
  case I: return mf_bits_kernel<KT, G, P>;
    MF_BITS_TABLE(MF_BITS_CASE)
#undef MF_BITS_CASE
    default: return nullptr;
  }
}

template <int KT>
BatchKernelFn pick_bits_batched_variant(int v) {
  switch (v) {
#define MF_BITS_CASE(I, G, P) \
  case I: return mf_bits_batched_kernel<KT, G, P>;
    MF_BITS_TABLE(MF_BITS_CASE)
#undef MF_BITS_CASE
    default: return nullptr;
  }
}

}  // namespace mf
