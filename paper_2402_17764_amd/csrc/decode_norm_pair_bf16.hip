// The decode kernel for bf16 x: RMSNorm in front, gate | up matrix, SwiGLU behind.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<true, true, true>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
