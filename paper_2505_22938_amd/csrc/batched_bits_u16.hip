// Batched bit-plane kernels for uint16 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
BatchKernelFn pick_bits_batched_u16(int v) { return pick_bits_batched_variant<KEY_U16>(v); }
}  // namespace mf
