// Bit-plane kernels for uint16 keys (bits_kernels.h).
#include "bits_kernels.h"

namespace mf {
PlainKernelFn pick_bits_u16(int v) { return pick_bits_variant<KEY_U16>(v); }
}  // namespace mf
