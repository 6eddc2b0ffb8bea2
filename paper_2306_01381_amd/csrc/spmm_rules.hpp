// Arithmetic of the sliced aggregation that host and device have to agree on, without HIP: a host compiler can check it.
#pragma once

#include <stdint.h>

namespace adaqp {

// Offset of a fetch that is to read nothing: past the end of any buffer the sliced kernel is launched with, also with a
// column offset (at most 8 KB) added.
constexpr uint32_t kOutside = 0xFFFF0000u;

// Bytes of a matrix of n_cols rows from column `begin` of its first row on: the extent of a buffer that starts there.
// Nothing where there are no rows: the difference would wrap to an extent that holds kOutside.
constexpr uint32_t buffer_extent(int64_t n_cols, int64_t ldh, int32_t begin)
{
    const int64_t floats = n_cols * ldh - begin;
    return floats > 0 ? (uint32_t)(floats * 4) : 0u;
}

// Whether the sliced kernel takes a launch.  Offsets of rows of H and of packed rows are kept in 32 bits.  Without columns or
// without entries there is nothing to gather and H, col and val may be NULL: the merge-path kernel then reads none of them,
// while the sliced one has loads in flight from the start.
constexpr bool sliced_takes(int64_t nnz, int64_t n_cols, int64_t ldh, bool packed, int64_t packed_bytes, int32_t full_dim)
{
    constexpr int64_t limit = (int64_t)kOutside;
    return nnz > 0 && n_cols > 0 && n_cols <= INT32_MAX && ldh < limit / 4 && n_cols * ldh < limit / 4 &&
           (!packed || packed_bytes < limit) && full_dim < (1 << 28);
}

}  // namespace adaqp
