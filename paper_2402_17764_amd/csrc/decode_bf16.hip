// The decode kernel for bf16 x: quantized as it is.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<true, false, false>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
