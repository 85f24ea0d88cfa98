// The decode kernel for bf16 x: gate | up matrix, SwiGLU behind.
#include "decode_kernel.hpp"

namespace bitnet {
template hipError_t launch_decode<true, false, true>(const DecodeForm&, const DecodeCall&);
}  // namespace bitnet
