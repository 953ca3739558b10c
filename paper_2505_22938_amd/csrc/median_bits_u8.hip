// Bit-plane kernels for uint8 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
PlainKernelFn pick_bits_u8(int v) { return pick_bits_variant<KEY_U8>(v); }
}  // namespace mf
