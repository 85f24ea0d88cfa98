// Where the 16-byte pieces of a row-major byte matrix are read from when its rows have any length.  Integer arithmetic only, so
// that it compiles for the device and, without HIP, for a test on the host.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define BITNET_BOTH __host__ __device__
#else
#define BITNET_BOTH
#endif

namespace bitnet {

// Pieces at offsets from byte `first` of the matrix on, `left` bytes to its end.  A piece that would run out of the matrix is pulled
// back: read from the last 16 bytes, and moved down by moved() to where it belongs.  A matrix of less than 16 bytes is not whole():
// it has no such piece.
struct ByteSpan {
    int lead, bytes;                                     // the span starts `lead` bytes in front of `first`
    BITNET_BOTH constexpr ByteSpan(int64_t first, int64_t left)
        : lead(first >= 16 ? 16 : 0),                    // so that 16 bytes precede the end
          bytes((int)(left + (first >= 16 ? 16 : 0) < 1 << 30 ? left + (first >= 16 ? 16 : 0) : 1 << 30)) {}
    BITNET_BOTH constexpr bool whole() const { return bytes >= 16; }
    BITNET_BOTH constexpr int at(int off) const { return lead + off < bytes - 16 ? lead + off : bytes - 16; }
    BITNET_BOTH constexpr int moved(int off) const { return lead + off - at(off); }
    // Whether a tile of `rows` rows of K bytes from `first` on has a piece that is pulled back.  Its last row's last piece is the
    // furthest one, and pieces of earlier K steps of 256 bytes end in front of their row's end.  The tile need not be the matrix's
    // last: with K below 16 a piece reaches over several rows, into and past the few that may follow.
    BITNET_BOTH constexpr bool pulls_back(int rows, int K) const { return moved((rows - 1) * K + ((K + 255) / 256 - 1) * 256 + 240) > 0; }
};

}  // namespace bitnet
