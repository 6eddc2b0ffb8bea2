// Internal helpers shared by the translation units of libadaqp (host side only, plus a few wave intrinsics).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "adaqp.h"

namespace adaqp {

// Records the text of a failed HIP call for adaqp_last_hip_error() and maps it to ADAQP_EHIP.
int note_hip_error(hipError_t err, const char *what);

#define ADAQP_HIP_TRY(expr)                                              \
    do {                                                                 \
        hipError_t adaqp_err__ = (expr);                                 \
        if (adaqp_err__ != hipSuccess) return ::adaqp::note_hip_error(adaqp_err__, #expr); \
    } while (0)

#define ADAQP_TRY(expr)                                                  \
    do {                                                                 \
        const int adaqp_rc__ = (expr);                                   \
        if (adaqp_rc__ != ADAQP_OK) return adaqp_rc__;                   \
    } while (0)

// adaqp_spmm_csr_packed (slot_of_row_dev NULL: adaqp_spmm_csr) with what the caller knows about the columns: skewed_columns
// = a few columns hold most of the entries, as in a transposed graph of power-law degrees, whose columns are used as often as
// their nodes' degrees say.  It only picks how the work is cut.
int spmm_rows(const int64_t *rowptr_dev, const int32_t *col_dev, const float *val_dev, int64_t nnz, int64_t row_begin,
              int64_t row_end, int64_t nnz_range, const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
              float *out_dev, int64_t ldo, const int32_t *slot_of_row_dev, const uint8_t *packed_dev,
              int64_t packed_bytes, const float *params_dev, const uint8_t *bits_dev, const int64_t *row_offset_dev,
              int64_t n_slots, void *workspace_dev, int64_t workspace_bytes, void *stream, bool skewed_columns);

// What adaqp_spmm_csr_segments and adaqp_spmm_csr_blocks refuse, but for their workspaces: the layer step asks before it queues anything.
int check_segments_call(const adaqp_spmm_segments *p, const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim, const float *out_dev,
                        int64_t ldo);
int check_blocks_call(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const float *H_dev, int64_t n_cols, int64_t ldh,
                      int32_t dim, const float *out_dev, int64_t ldo);

inline bool valid_bits(int b) { return b == 2 || b == 4 || b == 8; }

inline bool aligned_to(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

constexpr int kWave = 64;            // gfx950 wavefront width
constexpr int kBlock = 256;          // threads per workgroup used by every kernel here (4 waves)
constexpr int kWavesPerBlock = kBlock / kWave;

}  // namespace adaqp
