// The decode kernel for fp32 x: RMSNorm in front.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<false, true, false>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
