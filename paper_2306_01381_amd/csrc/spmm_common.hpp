// Shared by the aggregation kernels of spmm.hip and spmm_sliced.hip: the launch arguments and small device helpers.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "loop_back.hpp"
#include "spmm_rules.hpp"

namespace adaqp {

// Rows of H that are still packed (received halo rows, de-quantised on the fly).
struct PackedRows {
    const int32_t *slot_of_row; // [n_cols], -1 = read the row from H; NULL: no row is packed
    const uint8_t *packed;
    int64_t packed_bytes;
    const float *params;
    const uint8_t *bits;
    const int64_t *row_offset;
    int64_t n_slots;
    int32_t col0, full_dim;     // first column of this launch's chunk and the row length of the packed layout
    const adaqp_packed_row *row;        // [n_cols], planned pieces: in place of slot_of_row, bits and row_offset
};

struct SpmmArgs {
    const int64_t *rowptr;      // already offset: rowptr[0] is the start of the first row of the range
    const int32_t *col;
    const float *val;
    int64_t nnz;                // capacity of col / val
    int32_t n_rows;             // rows in the range
    const float *H;
    int64_t n_cols, ldh;
    int32_t dim, wdim;          // wdim >= dim: columns [dim, wdim) of a written row receive zeros (whole lines)
    float *out;                 // already offset to the first row of the range
    int64_t ldo;
    int32_t *carry_row;         // [n_items]
    float *carry;               // [n_items, carry_ld]
    int64_t carry_ld;
    int32_t n_items;
    PackedRows p;
};

__device__ __forceinline__ int64_t clamp64(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// The rows of a range with the feature columns sliced over the XCDs (spmm_sliced.hip).  plan_sliced: how, or lines = 0 where
// spmm_merge_kernel has to take the launch or is faster; nnz_hint is what the caller says of the entries.  launch_sliced uses
// a.n_items carry slots at most and writes how many are in use.
SlicedCut plan_sliced(const SpmmArgs &a, int64_t nnz_hint, bool whole_lines, bool skewed_columns);
hipError_t launch_sliced(const SpmmArgs &a, const SlicedCut &cut, int64_t nnz_hint, bool whole_lines, hipStream_t st,
                         int32_t *n_carries_out);

// Segments in planned pieces (spmm_pieces.hip): ptr, entries and destinations of n_seg segments, n_rows rows of out.
struct PieceArgs {
    const adaqp_spmm_piece *pieces;     // [n_pieces + 1]
    const int32_t *dest;                // [n_seg]
    const int64_t *ptr;                 // [n_seg + 1]
    const int32_t *col;
    const float *val;
    int64_t n_entries;                  // capacity of col / val
    int64_t n_walked;                   // of rows: entries that the caller says they have
    int32_t n_pieces, n_seg;
    bool of_rows;                       // segments are the rows of out (always where rows of H may be packed)
    const float *H;
    int64_t n_cols, ldh;
    PackedRows p;
    int32_t dim, wdim, lines;           // of a launch: columns, columns in whole lines, lines
    float *out;
    int64_t ldo;
    int32_t n_rows;
    float *partial;                     // [n_partials, ldp]
    int64_t ldp;
    int32_t n_partials;
    int32_t n_blocks;                   // workgroups per slice
    uint32_t copy_blocks;               // first workgroups of the launch, whole rounds over the XCDs, that copy, where rows may be packed
    LoopBack copies;
};
// What of a plan can be seen from the host, and the launches; the caller has filled in everything from ptr on but what the plan says.
int check_pieces(const adaqp_spmm_pieces *p, int64_t n_seg);
int launch_pieces(const adaqp_spmm_pieces *p, PieceArgs a, hipStream_t st);

}  // namespace adaqp
