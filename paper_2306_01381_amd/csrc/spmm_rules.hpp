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

// Row ends that one step of the search for a share's first row looks at (a wave, four each).  The search counts rows in 32
// bits, up to a step past the range.
constexpr int32_t kProbes = 256;

// Whether the sliced kernel takes a launch.  Offsets of rows of H and of packed rows are kept in 32 bits.  Without columns or
// without entries there is nothing to gather and H, col and val may be NULL: the merge-path kernel then reads none of them,
// while the sliced one has loads in flight from the start.
constexpr bool sliced_takes(int64_t n_rows, int64_t nnz, int64_t n_cols, int64_t ldh, bool packed, int64_t packed_bytes, int32_t full_dim)
{
    constexpr int64_t limit = (int64_t)kOutside;
    return n_rows + n_rows / kProbes + kProbes <= INT32_MAX && nnz > 0 && n_cols > 0 && n_cols <= INT32_MAX && ldh < limit / 4 && n_cols * ldh < limit / 4 &&
           (!packed || packed_bytes < limit) && full_dim < (1 << 28);
}

constexpr int kXcds = 8;

// How the sliced kernel cuts a launch: lines per slice for plain rows and where rows may still be packed, workgroups (of four
// shares) per slice.  lines 0: the merge-path kernel is the faster one.  n_blocks alone decides the order of additions and is
// the same for both: packed rows give the bits of the same rows de-quantised beforehand.
struct SlicedCut { int32_t lines, packed_lines; int64_t n_blocks; };

// Times below: merge-path kernel / sliced kernel, power-law columns, plain (packed) rows, measured over 3 750 to 450 000
// columns, 4 to 300 entries per row, 16 to 602 columns of H.
constexpr SlicedCut sliced_cut(int64_t n_rows, int64_t nnz, int64_t n_cols, int32_t lines, bool whole_lines, bool skewed_columns)
{
    constexpr int64_t kBlocks = 512;        // two workgroups on each CU
    constexpr SlicedCut kMergePath = {0, 0, 0};
    const int64_t degree = nnz / n_rows, fours = (lines + 3) / 4;
    // few entries: a share's search and the empty ring cost more than its entries (45 000 entries 0.8-1.0, 112 000 1.05-1.25;
    // whole slices of wide rows 80 000 1.1-1.2; a line left over 112 000 0.9, 180 000 1.1)
    const bool whole_fours = whole_lines && lines >= 12 && lines % 4 == 0, one_over = lines >= 9 && lines % 4 == 1;
    if (nnz < (whole_fours ? 60000 : (one_over ? 150000 : 100000))) return kMergePath;
    if (!whole_lines) {
        // rows that share lines: a slice of four lines touches five, and a row end costs more.  Rows up to two lines wide: 1.1-4.
        // Wider ones have to be long (18 entries x 300 columns 0.9-1.0), and past four lines what the slices keep in the L2s
        // has to be most of the columns (130 to 515 columns wide: 15 000 columns 1.1-1.5, 60 000 0.77-1.04)
        const bool pays = lines <= 2 ||
                          (degree >= 64 && (lines <= 4 || n_cols <= 30000 || (lines >= 16 && n_cols <= 100000)));
        return pays ? SlicedCut{4, 4, kBlocks / fours} : kMergePath;
    }
    // Lines per slice.  With four, one LDS read, one address and one row end serve four loads; with one, an L2 holds four times
    // as many rows: one pays where rows are long and the columns too many for an L2 to hold four lines of each (measured break-even
    // at 224 columns of H: 12 entries x 50 000 columns, 20 x 34 000, 40 x 20 000).  Where a few columns hold most of the
    // entries four lines of those fit anyway: transposed graph, power-law degrees, 150 000 columns, 30 entries per row, 256 columns of
    // H four lines 1.27, one 0.98.  (The caller says so by the direction; log-normal degrees there 1.11, 1.43.)
    const bool many = !skewed_columns && n_cols > 10240 && degree * n_cols > 700000;
    if (!many) {
        // rows of four or five entries: only where no slice is a line or three wide (160 columns 0.8-0.9, 352 columns packed 0.8)
        if (degree < 6 && lines >= 5 && lines % 2 == 1) return kMergePath;
        // two lines per slice where four would leave two over (300 columns: 1.3 against 1.1), or five lines as 4 + 1 (1.25, 1.0)
        const int32_t v = lines % 4 == 2 || lines == 5 ? 2 : 4;
        int64_t n_blocks = kBlocks / ((lines + v - 1) / v);
        // three lines over: the XCDs that take them have more tasks than room for workgroups, and twice as many of half the
        // size spread that (60 000 columns, 352 wide packed 1.03, 1.16; 602 wide 0.96, 1.15) where shares stay long enough
        // and the columns do not fit the L2s anyway (15 000 columns, 352 wide 1.7, 1.5)
        if (lines % 4 == 3 && lines >= 7 && (lines >= 15 || n_cols > 40000) && nnz >= 500 * 4 * 2 * n_blocks) n_blocks *= 2;
        return {v, v, n_blocks};
    }
    // Two per slice: past 200 000 columns, six times what an L2 holds of one line each, if lines come in pairs (plain rows
    // 1.02-1.2; one line 0.95-1.15).  Packed rows prefer four lines, whose codes share a line: with the same shares where the
    // lines come in fours (256 columns 0.95, 1.02; but 192 columns 1.05, 0.9), and wide ones with more shares (512 columns 0.92-1.0
    // against 0.80-0.93), which plain rows take without loss if they are 1 900 entries long and more than eight lines wide.
    if (n_cols > 200000 && lines % 2 == 0) {
        if (lines >= 10 && nnz >= 1900 * 4 * (2 * kBlocks / fours)) return {2, 4, 2 * kBlocks / fours};
        return {2, lines % 4 == 0 ? 4 : 2, kBlocks / (lines / 2)};
    }
    if (degree < 6 && lines >= 5) return kMergePath;        // (150 000 rows of four entries: 0.90-0.97)
    // one per slice, up to eight workgroups per CU in all; packed rows four (352 columns 1.2 against 0.8 with one)
    const bool halves = lines >= 5 && n_cols > 40000 && nnz >= 600 * 4 * (2 * kBlocks / fours);
    return {1, 4, (halves ? 2 : 1) * kBlocks / fours};
}

// Whether workgroups of the merge path add up the parts that their pieces have of a row.  That saves three of four carries and shortens the chain of
// a long row's, but the rows that begin a piece are stored a barrier and three LDS reads later, which launches of little else show.  A carry
// per piece / joined, 924 calls of two degree laws: rows of 10 and more entries 1.0-1.35 (mostly 1.02-1.25); of 1 to 4 entries, up to 5 000 rows
// 0.88-0.98, 150 000 rows of 301 columns 1.02-1.09, of 33 columns 1.0; of 6 entries 0.96 (log-normal degrees) and 1.08 (Zipf).
constexpr bool merge_joins(int64_t n_rows, int64_t nnz, int64_t n_items, int32_t dim)
{
    return nnz >= 6 * n_rows || n_items * dim >= 300000;
}

// Which workgroup takes which slice and share.  Tasks in slice-major order, n_blocks of each slice; consecutive workgroups land
// on consecutive XCDs, and an XCD takes a run of tasks of an eighth of the whole weight.  The last slice may be narrower than
// the others; walking the entries costs it as much as them, so a task weighs its lines and that walk.
struct SliceTasks {
    int64_t full, all;                  // tasks of whole slices; weight of all tasks
    int32_t whole_weight, rest_weight;  // of a task of a whole slice, of the narrower one (0: there is none)

    constexpr SliceTasks(int32_t lines, int32_t lines_per_slice, int32_t n_blocks, bool packed)
        : full((int64_t)(lines / lines_per_slice) * n_blocks), all(0), whole_weight(0), rest_weight(0)
    {
        // The walk is worth half a line of plain rows (160 columns in slices of four: 1.3 times as fast as with none, five
        // lines' worth 1.26; but seven lines 0.96), three lines where slots are looked up as well (288 to 519 columns 1.25-1.3)
        const int32_t rest = lines % lines_per_slice, walk = packed ? 6 : (rest == 3 ? 0 : 1);
        whole_weight = 2 * lines_per_slice + walk;
        rest_weight = rest ? 2 * rest + walk : 0;
        all = full * whole_weight + (int64_t)n_blocks * rest_weight;
    }

    // first task that begins at or after this much weight
    constexpr int64_t task_at(int64_t at) const
    {
        return at <= full * whole_weight || rest_weight == 0 ? (at + whole_weight - 1) / whole_weight
                                                             : full + (at - full * whole_weight + rest_weight - 1) / rest_weight;
    }
    constexpr int64_t first_task(int32_t xcd) const { return task_at(all * xcd / kXcds); }
    constexpr int64_t most_per_xcd() const          // what the grid has to provide for
    {
        int64_t most = 0;
        for (int32_t x = 0; x < kXcds; ++x)
            if (first_task(x + 1) - first_task(x) > most) most = first_task(x + 1) - first_task(x);
        return most;
    }
};

// What segments cost beside a walk over the rows, in entries times lines: the walk over all entries and a partial row and its sum per
// row.  Forward slices are one line, backward ones four: the weights differ.  (Fitted to steps timed with and without segments,
// adaqp_spmm_segments_gain.)
constexpr double segments_cost(bool transposed, double lines, double entries, double rows)
{
    return transposed ? (0.26 * lines + 0.41) * entries : (0.5 * lines + 0.25) * entries + 2.7 * lines * rows;
}

// What the matrix cores save of that for the entries of their rows, in forward steps.  They cost their coefficients once, however few lines
// there are: 50 000 rows, 97 entries per row, 64 columns 121 -> 151 us with segments and blocks; 60 000 rows, 110, 256 columns 525 -> 402.
constexpr double blocks_gain(double lines, double dense_entries) { return 0.56 * (lines > 1.5 ? lines - 1.5 : 0.0) * dense_entries; }

// Pieces of a plan, at most.
constexpr int64_t kMostPieces = 1 << 24;

// Lines that one launch of planned pieces takes at most, for n_blocks workgroups of so many waves per slice.  A launch has fewer than 2^32
// threads, and the grid has room for up to three times as many tasks as there are (SliceTasks: those of a narrower slice weigh that
// much less).
constexpr int64_t pieces_lines(int64_t n_blocks, int32_t waves, int32_t lines_per_slice)
{
    const int64_t slices = kMostPieces / waves / n_blocks;
    return (slices > 1 ? slices : 1) * lines_per_slice;
}

}  // namespace adaqp
