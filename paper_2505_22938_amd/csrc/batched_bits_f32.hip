// Batched bit-plane kernels for float32 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
BatchKernelFn pick_bits_batched_f32(int v) { return pick_bits_batched_variant<KEY_F32>(v); }
}  // namespace mf
