// The decode kernel for fp32 x: RMSNorm in front, gate | up matrix, SwiGLU behind.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<false, true, true>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
