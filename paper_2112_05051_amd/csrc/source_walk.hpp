// Limits of the 32-bit source lists that the hierarchy refresh sums
// (k_gal_sum), shared with a CPU check of them.  Plain C++ (no HIP).
#pragma once

#include <cstdint>

namespace rich {

// A block of the sum walks its stretch of the list, places [t0, t1), in pieces.
constexpr int GS_TPB = 256, GS_PER = 6, GS_PIECE = GS_TPB * GS_PER;

// Whether lists of nnz places, indexing arrays of `values` values, keep to 32
// bits.  A walk's last step, to at most t1 - 1 + GS_PIECE, must not wrap to the
// front: it would start over and never end.
inline bool source_lists_fit(int64_t nnz, int64_t values) {
    return nnz <= ((int64_t)1 << 32) - GS_PIECE && values <= (int64_t)1 << 32;
}

}  // namespace rich
