// Bit-plane kernels for float32 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
PlainKernelFn pick_bits_f32(int v) { return pick_bits_variant<KEY_F32>(v); }
}  // namespace mf
