// The decode kernel for bf16 x: RMSNorm in front.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<true, true, false>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
