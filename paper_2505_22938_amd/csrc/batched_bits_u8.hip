// Batched bit-plane kernels for uint8 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
BatchKernelFn pick_bits_batched_u8(int v) { return pick_bits_batched_variant<KEY_U8>(v); }
}  // namespace mf
