// The decode kernel for fp32 x: quantized as it is.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<false, false, false>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
