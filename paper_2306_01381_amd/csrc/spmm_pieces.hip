// Neighbour aggregation (Sec. 2.1 Eq. 3) over a planned walk: the segments of rows in the order of column tiles, cut into pieces by the
// host.  A wave takes one piece for one slice of VPL lines of H and gathers as spmm_sliced.hip does: one load per line for eight
// entries, AHEAD steps of eight in flight, sums folded over the eight groups where a segment ends.
//
// What bounds the gathers of segments is what their group of tiles misses in the L2, and that hangs on how far apart the entries are
// that an XCD has under way.  Shares cut on the device are a search each (eight loads that wait for one another, 20 us under load)
// and so have to be long: 128 workgroups with 4 600 entries each span two groups, 6 and 13 % of the lines of the two ranges of the step
// below come from behind the L2, and the L1, which answers in order, stands still for each of them (25 and 30 % of its time).  A planned
// piece begins with one load of its bounds and is 700 entries long; workgroups start in order, so that those under way are
// neighbours: 6 and 8 % from behind the L2, 17 and 23 %.
// Waves that take piece after piece drift apart and lose that (28 % from behind the L2, 1.29 -> 1.55 ms for the step below).
// A piece is one LDS fill, so nothing of the next has to wait in registers: 76 of them for segments, and no spilled scalars.
//
// 58 000 rows, 27.8 M entries, 98 000 columns, 256 columns of H, the whole layer step: shares 1.40 ms, here with as many waves as
// registers allow 1.29, with 16 per CU 1.19 (25 TB/s of gathers; bare loads out of the L2 31; 24 waves of two lines ask for more
// than their group; two lines per slice 1.19, one 1.46, four 1.31).  306 000 rows, 7.7 M entries, 456 000 columns, whose groups
// are three times an L2: shares 1.04 ms, two lines per slice 0.83, one 0.75.
#include <algorithm>
#include <cmath>
#include <functional>
#include <numeric>
#include <new>
#include <vector>

#include "spmm_common.hpp"
#include "spmm_wave.hpp"

namespace adaqp {
namespace {

constexpr int kEntries = ADAQP_SPMM_PIECE_ENTRIES, kFewEntries = 256;      // of a piece
constexpr int kJoinWaves = 8;                               // of a workgroup whose waves join the parts of a segment
constexpr int kEnds = ADAQP_SPMM_PIECE_SEGMENTS;
constexpr int kPart = 256;                                  // no sum runs longer than a part's 32 steps
constexpr int32_t kJoined = -2, kNowhere = INT32_MIN;       // a piece's partial; a destination
constexpr int32_t kMoved = INT32_MIN + 1;                   // in place of a destination: rowptr is no longer what the plan was made from
constexpr int32_t kNoEnd = 0x10000;                         // lies after every step of a piece
constexpr unsigned kIdleLds[2] = {6144, 24576};             // of a workgroup, beside its 26 KB: no more than 16 or 12 waves on a CU
constexpr unsigned kIdleLdsPacked = 12288;                  // beside 52 KB: 8 instead of 12
static_assert(kEnds < kWave - 1, "a lane per end, and one that has none");

// A sum to its place.  Lanes without a column of their own store outside the row's buffer: no branch.
template <int VPL>
__device__ __forceinline__ void store_row(const PieceArgs &a, float *row, bool known, int32_t first_line, int lane, const float (&sum)[VPL])
{
    const uint32_t at = lane < kLine ? (uint32_t)(first_line * kLine + lane) * 4u : kOutside;
    const auto to = __builtin_amdgcn_make_buffer_rsrc(row, 0, known ? a.wdim * 4 : 0, kRawBuffer);
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const float x = (first_line + v) * kLine + (lane & (kLine - 1)) < a.dim ? sum[v] : 0.0f;        // row padding
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), to, (int)at + v * kLine * 4, 0, kNonTemporal);
    }
}

// dest: a partial row, or -1 - row.
template <int VPL>
__device__ __forceinline__ void store_row(const PieceArgs &a, int32_t dest, int32_t first_line, int lane, const float (&sum)[VPL])
{
    const bool part = dest >= 0, known = part ? dest < a.n_partials : -1 - dest < a.n_rows;
    store_row<VPL>(a, part ? a.partial + (int64_t)dest * a.ldp : a.out + (int64_t)(-1 - dest) * a.ldo, known, first_line, lane, sum);
}

// An entry in LDS.  Where rows may be packed: its place rotated by two, so that the width of a packed row is at the top and the row's 32-bit word in
// the others; not what Entry<true> holds, which keeps the width in the lowest bits.
struct alignas(16) RotatedEntry { uint32_t place; float val; float z, s; };
static_assert(!std::is_convertible_v<Entry<true>, RotatedEntry> && !std::is_convertible_v<RotatedEntry, Entry<true>>,
              "unpack_lines and unpack_codes read places of their own kind only");
template <bool PACKED> using PieceEntry = std::conditional_t<PACKED, RotatedEntry, Entry<false>>;

__device__ __forceinline__ uint32_t packed_width(const RotatedEntry &en) { return en.place >> 30; }

// Byte offset of the row in H.
__device__ __forceinline__ uint32_t row_offset(const RotatedEntry &en) { return en.place << 2; }
__device__ __forceinline__ uint32_t row_offset(const Entry<false> &en) { return en.off; }

// unpack_codes of a lane's columns in VPL lines: a line's codes fill whole words at each width, so they begin at the same bit in all of
// them, and v_bfe_u32 takes that modulo 32 by itself.  Where most rows come out of the L2 the instructions count: with these places, one shift
// per entry and the words asked for before the rows, 24 000 rows of 17 entries, 66 columns, packed, the step 30.1 -> 28.4 us; 7 700 of 156, 316
// columns 131 -> 109; 17 500 of 75, 96 columns 66 -> 54; 150 such steps 1.055 times as fast.
template <int VPL>
__device__ __forceinline__ void unpack_lines(const RotatedEntry &en, const uint32_t (&words)[VPL], uint32_t col, float4_t (&x)[VPL])
{
    const uint32_t w = packed_width(en);
    const uint32_t b = 1u << w, at = col << w;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        if (w == 0) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float scaled = (float)__builtin_amdgcn_ubfe(words[v], at + k * b, b) * en.s;
            x[v][k] = scaled + en.z;
        }
    }
}

// stage_entries where rows may be packed, whose places have been looked up beforehand: a load per entry and one of (Z, S) instead of four, and
// two that wait for one another instead of three (24 000 rows, 0.42 M entries, 66 columns, whole step: 40.2 -> 37.4 us; shares cut on the
// device 38.7).
template <int LOADS>
__device__ __forceinline__ void stage_packed(int4_t (&st_col)[LOADS], const float4_t (&st_val)[LOADS], int32_t n_ent, uint32_t n_cols,
                                             uint32_t pitch, const PackedRows &p, int lane, RotatedEntry *stage)
{
    auto valid = [&](int k, int q) ADAQP_INLINE { return (k * kWave + lane) * 4 + q < n_ent && (uint32_t)st_col[k][q] < n_cols; };
    uint2 at[LOADS][4];
#pragma unroll
    for (int k = 0; k < LOADS; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) at[k][q] = *reinterpret_cast<const uint2 *>(p.row + (valid(k, q) ? st_col[k][q] : 0));
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        if (k > 0 && k * 4 * kWave >= n_ent) break;         // a whole number of turns past every entry: never read
        bool packed[4];
        float2 zs[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            packed[q] = valid(k, q) && at[k][q].x != 0 && at[k][q].y < (uint64_t)p.n_slots;
            zs[q] = *reinterpret_cast<const float2 *>(p.params + 2 * (int64_t)(packed[q] ? at[k][q].y : 0));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t row = valid(k, q) ? (uint32_t)st_col[k][q] * pitch : kOutside;
            stage[(k * kWave + lane) * 4 + q] = RotatedEntry{__builtin_rotateright32(packed[q] ? at[k][q].x : row, 2),
                                                             valid(k, q) ? st_val[k][q] : 0.0f, zs[q].x, zs[q].y};
        }
    }
}

// What the waves of a workgroup hand to each other: lane l has column l of each line.
struct Joined {
    float open[4][kWave];       // the wave's part of the segment that its piece leaves open
    float first[4][kWave];      // its part of the first segment that ends in its piece, where other waves have parts of that
};

// A piece of rows whose rowptr was written to after it was planned, for all `live` lines of a slice.  The wave adds up what its piece is due of
// each of its rows: the entries of the row as they are now, from where the piece begins if it was planned to begin inside the row, up
// to where it ends if it was planned to end inside.  The pieces of a row so have each of its entries once, wherever it lies.  Returns
// what walk_piece does.  No limit to how long a row can have become: one line at a time, no staging, few registers.  What bounds it is the
// piece that has become the longest (lengths of the rows permuted, the whole step as planned, so, and cut on the device: 2 000 rows, 128
// columns 13, 35, 19 us; 24 000 rows, 66 columns, packed 28, 720, 46; 376 000 rows, 256 columns 0.84, 5.0, 0.86 ms, with 16 waves per CU 4.1).
template <bool PACKED, bool JOINS>
__device__ __forceinline__ int32_t walk_moved(const PieceArgs &a, const int32_t first_line, const int live, const int32_t item, Joined *joined)
{
    constexpr int kAhead = 4;                               // steps on their way
    const int lane = threadIdx.x & (kWave - 1), gl = lane & (kGroup - 1), grp = lane / kGroup;
    const adaqp_spmm_piece from = a.pieces[item], to = a.pieces[item + 1];
    const int32_t seg0 = min(max(from.segment, 0), a.n_seg);
    const int32_t n_end = min(max(to.segment - seg0, 0), min(a.n_seg - seg0, kEnds));
    const int32_t n_mine = min(n_end + (to.partial != -1 ? 1 : 0), a.n_seg - seg0);
    int32_t join_dest = kNowhere;
    for (int32_t q = 0; q < n_mine; ++q) {
        int64_t first = max(a.ptr[seg0 + q], (int64_t)0), end = min(a.ptr[seg0 + q + 1], a.n_entries);
        if (q == 0 && from.partial != -1) first = max(first, from.entry);
        if (q == n_end) end = min(end, to.entry);
        const int32_t dest = q < n_end ? a.dest[seg0 + q] : to.partial;
        for (int v = 0; v < live; ++v) {
            const int32_t at = (first_line + v) * kLine + gl * 4;
            const uint32_t packed_col = (uint32_t)(a.p.col0 + at);
            float4_t total = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int64_t part = first; part < end; part += kPart) {
                const int64_t part_end = min(end, part + kPart);
                float4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
                for (int64_t e0 = part; e0 < part_end; e0 += kAhead * kStep) {
                    float val[kAhead];
                    float4_t x[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int64_t e = min(e0 + u * kStep + grp, part_end - 1);
                        const int32_t c = a.col[e];
                        const bool ok = e0 + u * kStep + grp < part_end && (uint32_t)c < (uint32_t)a.n_cols;
                        const int64_t row = ok ? c : 0;
                        val[u] = ok ? a.val[e] : 0.0f;
                        x[u] = *reinterpret_cast<const float4_t *>(a.H + row * a.ldh + at);
#pragma unroll
                        for (int k = 0; k < 4; ++k) x[u][k] = ok ? x[u][k] : 0.0f;
                        if constexpr (PACKED) {
                            const adaqp_packed_row place = a.p.row[row];
                            if (ok && place.place != 0 && place.slot < (uint64_t)a.p.n_slots) {
                                const uint32_t w = place.place & 3u, last_word = (((uint32_t)a.p.full_dim << w) - 1) >> 5;
                                const uint32_t word = *reinterpret_cast<const uint32_t *>(
                                    a.p.packed + (place.place & ~3u) + 4 * (int64_t)min((packed_col << w) >> 5, last_word));
                                const float2 zs = *reinterpret_cast<const float2 *>(a.p.params + 2 * (int64_t)place.slot);
                                x[u] = unpack_codes(Entry<true>{place.place, val[u], zs.x, zs.y}, word, packed_col, x[u]);
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u)
#pragma unroll
                        for (int k = 0; k < 4; ++k) sum[k] = fmaf(val[u], x[u][k], sum[k]);
                }
                total += sum;
            }
            float sum[1] = {0.0f};                          // lane l: column l of the line, of all groups
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                for (int other = kGroup; other < kWave; other *= 2) total[k] += __shfl_xor(total[k], other);
                const float of_column = __shfl(total[k], (lane & (kLine - 1)) / 4);
                if ((lane & 3) == k) sum[0] = of_column;
            }
            if (JOINS && q == 0 && q < n_end && from.partial == kJoined) {
                join_dest = dest;
                joined->first[v][lane] = sum[0];
            } else if (JOINS && q == n_end && dest == kJoined) {
                joined->open[v][lane] = sum[0];
            } else if (q < n_end || dest >= 0) {
                store_row<1>(a, dest, first_line + v, lane, sum);
            }
        }
    }
    return join_dest;
}

// ROWS: segments are rows, whose sums go to one row after the other but for those with parts.  JOINS: parts of a segment may be other
// waves' of the workgroup.  Returns where the sum of such a segment goes that ends in this piece, kNowhere, or
// kMoved before anything is written (ROWS).
template <int VPL, int AHEAD, bool PACKED, bool ROWS, bool JOINS, int ENTRIES>
__device__ __forceinline__ int32_t walk_piece(const PieceArgs &a, const int32_t first_line, const int32_t item, PieceEntry<PACKED> *stage, Joined *joined)
{
    constexpr int kRing = AHEAD * kStep;                    // entries of a turn of the ring
    constexpr int kParts = ENTRIES / kPart;
    constexpr int kLoads = ENTRIES / (4 * kWave);           // of four entries per lane: what a piece takes of col, and of val
    static_assert(kPart % kRing == 0 && ENTRIES % kPart == 0 && kPart / kStep <= 32, "a part is a whole number of turns, a bit per step");
    const int lane = threadIdx.x & (kWave - 1), gl = lane & (kGroup - 1), grp = lane / kGroup;

    const adaqp_spmm_piece from = a.pieces[item], to = a.pieces[item + 1];
    const int32_t seg0 = min(max(from.segment, 0), a.n_seg);
    const int32_t n_end = min(max(to.segment - seg0, 0), min(a.n_seg - seg0, kEnds));
    const int64_t ent0 = clamp64(from.entry, 0, a.n_entries);
    const int32_t n_ent = (int32_t)clamp64(to.entry - ent0, 0, min((int64_t)ENTRIES, a.n_entries - ent0));
    // Steps are counted so that the last turn of the ring is a full one: a fetch of nothing takes as long as one of a line.  From the same
    // number on for every VPL, so that a part ends with the same entry and the sums are the same bits.
    const int32_t n_steps = (n_ent + kStep - 1) / kStep, pad = -n_steps & 7, first_turn = pad / AHEAD, turns = (n_steps + pad) / AHEAD;
    static_assert(8 % AHEAD == 0, "turns of eight steps or fewer");

    const auto cols = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(a.col + ent0), 0, n_ent * 4, kRawBuffer);
    const auto vals = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.val + ent0), 0, n_ent * 4, kRawBuffer);
    int4_t st_col[kLoads];
    float4_t st_val[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {                      // streamed: keep the caches for H; past the piece's entries: zeros
        const int at = (k * kWave + lane) * 16;
        st_col[k] = __builtin_bit_cast(int4_t, __builtin_amdgcn_raw_buffer_load_b128(cols, at, 0, kNonTemporal));
        st_val[k] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(vals, at, 0, kNonTemporal));
    }
    int32_t ends = kNoEnd, dests = -1;                      // lane l: where segment seg0 + l ends, and where its sum goes
    const bool open = ROWS && to.partial != -1;             // a row goes on in the next piece: lane n_end
    int64_t end = 0;
    if (lane < n_end + open) end = a.ptr[(int64_t)min(seg0 + lane + 1, a.n_seg)] - ent0;
    if (lane < n_end) {
        ends = (int32_t)clamp64(end, 0, n_ent) + pad * kStep;
        dests = a.dest[seg0 + lane];
    }
    if constexpr (ROWS) {                                   // the caller's rowptr, which may have been written to: still the rows of the plan?
        const int64_t begin = a.ptr[seg0] - ent0;
        bool moved = lane < n_end ? end < 0 || end > n_ent : open && lane == n_end && end < n_ent;
        moved |= lane == 0 && n_end + open > 0 && (from.partial == -1 ? begin != 0 : begin > 0);
        moved |= lane > 0 && ends < __shfl_up(ends, 1);
        if (__ballot(moved) != 0) return kMoved;
    }

    const uint64_t with_parts = __ballot(dests >= 0);
    float *out_row = a.out + (int64_t)seg0 * a.ldo;         // ROWS
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.H + first_line * kLine), 0,
                                                        (int)buffer_extent(a.n_cols, a.ldh, first_line * kLine), kRawBuffer);
    const auto packed_rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.p.packed), 0, (int)(uint32_t)a.p.packed_bytes, kRawBuffer);
    if constexpr (PACKED) stage_packed<kLoads>(st_col, st_val, n_ent, (uint32_t)a.n_cols, (uint32_t)a.ldh * 4u, a.p, lane, stage + pad * kStep);
    else stage_entries<kLoads, false>(st_col, st_val, n_ent, (uint32_t)a.n_cols, (uint32_t)a.ldh * 4u, a.p, lane, stage + pad * kStep);
    uint32_t marks[kParts];                                 // bit s: a segment ends in step s of the part, after one of its entries
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
        const int32_t last = ends - 1 - p * kPart;
        marks[p] = or_lanes(ends > pad * kStep && last >= 0 && last < kPart ? 1u << (last / kStep) : 0u);
    }

    // Sums of the open segment: acc what the present part has given so far, per group; before what earlier parts gave, lane l (and
    // l + 32) column l of each line.
    const int line_col = lane & (kLine - 1);
    const int from_lane = ((line_col & 3) * 16 + line_col / 4) << 2;
    float4_t acc[VPL];
    float before[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        before[v] = 0.0f;
    }
    auto take_sums = [&](float (&sum)[VPL]) ADAQP_INLINE {               // and start anew
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const float lo = fold<32>(acc[v][0], acc[v][2]), hi = fold<32>(acc[v][1], acc[v][3]);
            float x = fold<16>(lo, hi);                     // row q of 16 lanes: column 4 * gl + q, twice
            x = x + ror8(x);
            sum[v] = before[v] + __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from_lane, __builtin_bit_cast(int32_t, x)));
            before[v] = 0.0f;
            acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    auto to_lds = [&](float (&to)[4][kWave], const float (&sum)[VPL]) ADAQP_INLINE {
#pragma unroll
        for (int v = 0; v < VPL; ++v) to[v][lane] = sum[v];
    };

    // the ring: AHEAD steps whose lines are on their way
    float4_t h[AHEAD][VPL];
    uint32_t words[AHEAD][VPL];                             // of a packed row: the word that holds the lane's four codes
    PieceEntry<PACKED> in_flight[AHEAD];
    const uint32_t lane_off = gl * 16;
    const uint32_t packed_col = (uint32_t)(a.p.col0 + first_line * kLine + gl * 4);     // of the lane's codes in the first line
    const uint32_t last_col = min(packed_col + (VPL - 1) * kLine, (uint32_t)a.p.full_dim - 1);
    auto fetch = [&](auto tag, const PieceEntry<PACKED> &en) ADAQP_INLINE {
        constexpr int U = decltype(tag)::value;
        in_flight[U] = en;
        uint32_t off = row_offset(en) + lane_off;
        if constexpr (PACKED) {
            const uint32_t width = packed_width(en);
            off = width != 0 ? kOutside : off;
            // The word of the lane's four codes, and as far behind it the one of each line.
            const uint32_t first = width != 0 ? (en.place + (packed_col << width >> 5)) << 2 : kOutside;
            const uint32_t last = width != 0 ? (en.place + (last_col << width >> 5)) << 2 : kOutside;
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const uint32_t at = v + 1 < VPL ? first + ((uint32_t)v * (kLine / 8) << width) : last;
                words[U][v] = __builtin_amdgcn_raw_buffer_load_b32(packed_rows, (int)at, 0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            h[U][v] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(off + v * kLine * 4), 0, 0));
    };
    unroll<0, AHEAD>([&](auto tag) ADAQP_INLINE {
        constexpr int U = decltype(tag)::value;
        if (U >= pad % AHEAD) {
            fetch(tag, stage[(first_turn * AHEAD + U) * kStep + grp]);
        } else {
            in_flight[U] = {};
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                h[U][v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                words[U][v] = 0;
            }
        }
    });
    int32_t e = 0, join_dest = kNowhere;                    // segment ends behind us
    // One copy of the folds, whatever becomes of the sums: the kernel whose waves join parts has 79 registers, 95 with a copy for each place
    // (24 000 rows, 0.42 M entries, 66 columns, packed: the step 32.7 -> 32.3 us).
    auto end_segment = [&]() ADAQP_INLINE {
        float sum[VPL];
        take_sums(sum);
        if (JOINS && e == 0 && from.partial == kJoined) {
            join_dest = __builtin_amdgcn_readlane(dests, e);
            to_lds(joined->first, sum);
        } else if (ROWS) {
            float *row = out_row;
            bool known = true;
            if (with_parts >> e & 1) {
                const int32_t dest = __builtin_amdgcn_readlane(dests, e);
                row = a.partial + (int64_t)dest * a.ldp;
                known = dest < a.n_partials;
            }
            store_row<VPL>(a, row, known, first_line, lane, sum);
        } else store_row<VPL>(a, __builtin_amdgcn_readlane(dests, e), first_line, lane, sum);
        out_row += a.ldo;
        ++e;
    };
    while (__builtin_amdgcn_readlane(ends, e) <= pad * kStep) {      // segments without entries
        end_segment();
    }
    auto turn = [&](int32_t t, auto goes_on) ADAQP_INLINE {
        constexpr bool kGoesOn = decltype(goes_on)::value;  // else: the last one, whose lines are the last
        if (kParts > 1 && t > 0 && t % (kPart / kRing) == 0) {          // the next part
#pragma unroll
            for (int p = 0; p + 1 < kParts; ++p) marks[p] = marks[p + 1];
            float sum[VPL];
            take_sums(sum);
#pragma unroll
            for (int v = 0; v < VPL; ++v) before[v] = sum[v];
        }
        PieceEntry<PACKED> en[AHEAD];
        if constexpr (kGoesOn)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) en[u] = stage[(t + 1) * kRing + u * kStep + grp];
        __builtin_amdgcn_sched_barrier(0);
        unroll<0, AHEAD>([&](auto tag) ADAQP_INLINE {
            constexpr int U = decltype(tag)::value;
            float4_t x[VPL];
            float val = in_flight[U].val;
#pragma unroll
            for (int v = 0; v < VPL; ++v) x[v] = h[U][v];
            if constexpr (PACKED) unpack_lines<VPL>(in_flight[U], words[U], packed_col, x);
            if (marks[0] & (1u << U)) {
                // the groups from the last end to this one belong to the segment that ends here
                const int32_t at = (t * AHEAD + U) * kStep;
                int32_t first = 0, end = __builtin_amdgcn_readlane(ends, e) - at;
                do {
                    const bool mine = grp >= first && grp < end;
#pragma unroll
                    for (int v = 0; v < VPL; ++v)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float sum = fmaf(val, x[v][k], acc[v][k]);
                            acc[v][k] = mine ? sum : acc[v][k];
                        }
                    end_segment();
                    first = end;
                    end = __builtin_amdgcn_readlane(ends, e) - at;
                } while (end <= kStep);
                // what is left is the next segment's; no else: the sums would be copied where two branches meet
                val = grp >= first ? val : 0.0f;
#pragma unroll
                for (int v = 0; v < VPL; ++v)
#pragma unroll
                    for (int k = 0; k < 4; ++k) x[v][k] = grp >= first ? x[v][k] : 0.0f;
            }
#pragma unroll
            for (int v = 0; v < VPL; ++v)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[v][k] = fmaf(val, x[v][k], acc[v][k]);
            if constexpr (kGoesOn) fetch(tag, en[U]);
            __builtin_amdgcn_sched_barrier(0);
        });
        marks[0] >>= AHEAD;
    };
    marks[0] >>= first_turn * AHEAD;
    int32_t t = first_turn;
    for (; t + 1 < turns; ++t) turn(t, std::true_type());
    if (t < turns) turn(t, std::false_type());
    // of a segment that goes on in the next piece
    if (to.partial >= 0 || (JOINS && to.partial == kJoined)) {
        float sum[VPL];
        take_sums(sum);
        if (JOINS && to.partial == kJoined) to_lds(joined->open, sum);
        else store_row<VPL>(a, to.partial, first_line, lane, sum);
    }
    return join_dest;
}

template <int VPL, int AHEAD, bool PACKED, bool ROWS, int WAVES, int ENTRIES>
__global__ __launch_bounds__(WAVES * kWave, PACKED && ENTRIES > kFewEntries ? 2 : 4) void spmm_pieces_kernel(const PieceArgs a)
{
    constexpr bool kJoins = WAVES > kWavesPerBlock;
    __shared__ alignas(16) PieceEntry<PACKED> stages[WAVES][ENTRIES + kWave];
    __shared__ Joined joined[kJoins ? WAVES : 1];
    if constexpr (PACKED) if (blockIdx.x < a.copy_blocks) return copy_blocks(a.copies, blockIdx.x, WAVES * kWave);
    const uint32_t block = PACKED ? blockIdx.x - a.copy_blocks : blockIdx.x;
    const SliceTasks tasks(a.lines, VPL, a.n_blocks, PACKED);
    const int32_t xcd = block % kXcds;
    const int64_t task = tasks.first_task(xcd) + block / kXcds;
    if (task >= tasks.first_task(xcd + 1)) return;          // the whole workgroup
    const int32_t slice = (int32_t)(task / a.n_blocks), blk = (int32_t)(task % a.n_blocks), line = slice * VPL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t item = blk * WAVES + wave;
    const int live = min(VPL, a.lines - line);
    Joined *mine = joined + (kJoins ? wave : 0);
    int32_t dest = kNowhere;
    if (item < a.n_pieces) {
        if (live == VPL) dest = walk_piece<VPL, AHEAD, PACKED, ROWS, kJoins, ENTRIES>(a, line, item, stages[wave], mine);
        if constexpr (VPL > 3) if (live == 3) dest = walk_piece<3, AHEAD, PACKED, ROWS, kJoins, ENTRIES>(a, line, item, stages[wave], mine);
        if constexpr (VPL > 2) if (live == 2) dest = walk_piece<2, 2 * AHEAD, PACKED, ROWS, kJoins, ENTRIES>(a, line, item, stages[wave], mine);
        if constexpr (VPL > 1) if (live == 1) dest = walk_piece<1, 8, PACKED, ROWS, kJoins, ENTRIES>(a, line, item, stages[wave], mine);
        if constexpr (ROWS) if (dest == kMoved) dest = walk_moved<PACKED, kJoins>(a, line, live, item, mine);
    }
    if constexpr (kJoins) {
        __syncthreads();
        if (dest == kNowhere) return;
        const int lane = threadIdx.x & (kWave - 1);
        int from = wave;                                    // the wave whose piece the segment begins in
        const int32_t segment = a.pieces[item].segment;
        while (from > 0 && a.pieces[blk * WAVES + from].partial == kJoined && a.pieces[blk * WAVES + from].segment == segment) --from;
        for (int v = 0; v < live; ++v) {
            float sum[1] = {joined[from].open[v][lane]};
            for (int w = from + 1; w < wave; ++w) sum[0] += joined[w].open[v][lane];
            sum[0] += mine->first[v][lane];
            store_row<1>(a, dest, line + v, lane, sum);
        }
    }
}

// out[row] = sum of the row's partial rows, always in the same order; whole lines, row padding zero.  A wave per row and strip of at most
// 256 columns (28 000 rows of eight, 256 columns: 42 us, 6.1 TB/s).  Rows of one segment need none: of 306 000 rows one in twelve has
// two (129 -> 20 us).  Few rows are bound by the latency of their loads: narrow strips leave the wave's other lanes to other parts, and
// the strips of a wide row are waves of their own.  Sums go by pairs, as a chain of 24 parts is where the error of a long row comes from.
__global__ __launch_bounds__(kBlock) void pieces_sum_kernel(const int32_t *sum_row, const int32_t *sum_ptr, int64_t n_sums, int32_t n_partials,
                                                            const float *partial, int32_t dim, int64_t wdim, float *out, int64_t ldo, int32_t n_rows)
{
    constexpr int kAhead = 8;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t s = (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (s >= n_sums) return;
    const int32_t row = sum_row[s], from = max(0, sum_ptr[s]), end = min(sum_ptr[s + 1], n_partials);
    if (row < 0 || row >= n_rows) return;
    const int of_part = wdim <= 32 ? 8 : wdim <= 64 ? 16 : wdim <= 128 ? 32 : kWave;        // lanes of one part
    const int apart = kWave / of_part;
    for (int64_t strip = blockIdx.y; strip * kWave * 4 < wdim; strip += gridDim.y) {
        const int64_t c = (strip * kWave + lane % of_part) * 4;
        float4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int64_t p = from + lane / of_part; p < end; p += kAhead * apart) {
            float4_t x[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                x[q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                if (p + q * apart < end && c < wdim)
                    x[q] = __builtin_nontemporal_load(reinterpret_cast<const float4_t *>(partial + (p + q * apart) * wdim + c));
            }
#pragma unroll
            for (int half = kAhead / 2; half > 0; half /= 2)
#pragma unroll
                for (int q = 0; q < half; ++q) x[q] += x[q + half];
            sum += x[0];
        }
        for (int other = of_part; other < kWave; other *= 2)
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[k] += __shfl_xor(sum[k], other);
        if (lane >= of_part || c >= wdim) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k >= dim) sum[k] = 0.0f;
        __builtin_nontemporal_store(sum, reinterpret_cast<float4_t *>(out + (int64_t)row * ldo + c));
    }
}

// Length of a piece in entries and eight times ends of segments, the entries it has at most, waves of a workgroup.
//
// As many pieces as waves are under way, or half as many again where there are enough, but a start costs 0.2 us of its CU (28 M
// entries, 256 columns, two lines: 320 long 1.37 ms, 512 1.19, 864 1.19; 7.7 M entries, one line: 320 0.765, 448 0.753, 524 0.767;
// 1.2 M entries, 128 columns, four lines: 128 48 us, 220 45, 448 45).
//
// Where pieces are short anyway workgroups are twice as large and a segment's parts meet in their LDS: 2 000 rows, 20 656
// entries, 128 columns of H 7.2 us where 6.2 and a launch of sums of 3.3 (pieces of 96; 128 7.7, 16 waves and 128 8.9).
constexpr int64_t kUnderWay = 4096, kShort = 160;           // waves; a length

struct PieceShape { int64_t length, entries; int32_t waves; };

PieceShape piece_shape(int64_t n_seg, int64_t n_entries, int32_t dim, int32_t lines_per_slice)
{
    const int64_t slices = ((int64_t)dim + 32 * lines_per_slice - 1) / (32 * lines_per_slice);
    const double path = (double)(n_entries + 8 * n_seg) * (double)slices;
    if (path <= (double)(kUnderWay * kShort)) return {std::max<int64_t>((int64_t)path / kUnderWay, 96), kFewEntries, kJoinWaves};
    const int64_t most = lines_per_slice == 1 ? 448 : kEntries + 96;
    int64_t length = (int64_t)std::min(std::max(path / (1.5 * (double)kUnderWay), 128.0), (double)most);
    if (length <= kFewEntries + kFewEntries / 4) length = std::min<int64_t>(length, kFewEntries);       // for a third of the LDS and of the staging
    return {length, length <= kFewEntries ? kFewEntries : kEntries, kWavesPerBlock};
}

}  // namespace

int check_pieces(const adaqp_spmm_pieces *p, int64_t n_seg)
{
    if (p->n_pieces < 0 || p->n_partials < 0 || p->n_sums < 0 || n_seg < 0) return ADAQP_EINVAL;
    if (p->n_pieces == 0) return ADAQP_OK;
    if (p->n_pieces > kMostPieces || p->n_partials > INT32_MAX - 1024 || p->n_sums > INT32_MAX - 1024) return ADAQP_ESIZE;
    if (p->lines_per_slice != 1 && p->lines_per_slice != 2 && p->lines_per_slice != 4) return ADAQP_EINVAL;
    if (!(p->waves == kJoinWaves && p->entries == kFewEntries) && !(p->waves == kWavesPerBlock && (p->entries == kFewEntries || p->entries == kEntries)))
        return ADAQP_EINVAL;
    if (p->n_seg != n_seg || p->row_begin < 0) return ADAQP_EINVAL;
    if (!p->pieces_dev || !p->sum_ptr_dev || (n_seg > 0 && !p->dest_dev) || (p->n_sums > 0 && !p->sum_row_dev)) return ADAQP_EINVAL;
    if (!aligned_to(p->pieces_dev, 16) || !aligned_to(p->dest_dev, 4) || !aligned_to(p->sum_row_dev, 4) || !aligned_to(p->sum_ptr_dev, 4)) return ADAQP_EINVAL;
    return ADAQP_OK;
}

namespace {

using PieceKernel = void (*)(const PieceArgs);

template <bool PACKED, bool ROWS, int WAVES, int ENTRIES>
PieceKernel kernel_of(int32_t lines_per_slice)
{
    if constexpr (PACKED && ENTRIES == kEntries)
        if (lines_per_slice == 2) return spmm_pieces_kernel<2, 4, true, ROWS, WAVES, ENTRIES>;
    if constexpr (PACKED) return spmm_pieces_kernel<4, 2, true, ROWS, WAVES, ENTRIES>;
    else return lines_per_slice == 1   ? spmm_pieces_kernel<1, 8, false, ROWS, WAVES, ENTRIES>
                : lines_per_slice == 2 ? spmm_pieces_kernel<2, 4, false, ROWS, WAVES, ENTRIES>
                                       : spmm_pieces_kernel<4, 2, false, ROWS, WAVES, ENTRIES>;
}

template <bool PACKED, bool ROWS>
PieceKernel kernel_of(const adaqp_spmm_pieces *p, int32_t lines_per_slice)
{
    if (p->waves == kJoinWaves) return kernel_of<PACKED, ROWS, kJoinWaves, kFewEntries>(lines_per_slice);
    return p->entries == kFewEntries ? kernel_of<PACKED, ROWS, kWavesPerBlock, kFewEntries>(lines_per_slice)
                                     : kernel_of<PACKED, ROWS, kWavesPerBlock, kEntries>(lines_per_slice);
}

// Lines per slice where rows may be packed.  Their codes share lines, and each slice looks up the places again: four, but two where the plan
// says two and rows are shorter than 100 entries (four, two: 10 000 rows of 56 entries, 414 columns 88.7, 80.7 us; 15 000 of 47, 160 columns 56.6,
// 53.3; 27 000 of 19, 336 columns 90.7, 85.6; 11 000 of 67, 336 columns 97.9, 100.2; but 394 entries, 441 columns 121, 130; 298 entries, 208 columns
// 191, 197) and whole slices of four are not waves enough (157 000 rows, 240 columns, 4 600 waves: 175, 186).  80 steps of 9 to 150 entries per row,
// 160 to 600 columns, whose plan says two: where the rule takes two 0.94 to 1.28 times as fast, 1.07 on average, elsewhere 0.90 to 1.22.  In small
// pieces 0.94 to 1.03 with two; where the plan says one 0.89 to 1.12, four 0.89 to 1.04.  The same bits either way.
int32_t packed_lines(const adaqp_spmm_pieces *p, const PieceArgs &a, int64_t lines)
{
    const bool fills = lines % 4 == 0 && a.n_pieces * (lines / 4) >= kUnderWay;
    return p->lines_per_slice == 2 && p->entries == kEntries && lines > 4 && !fills && a.n_walked < 100 * (int64_t)a.n_seg ? 2 : 4;
}

// LDS that keeps waves away.  Where the L1 returns data all the time already (94 % of it, 16.3 M entries, 376 000 rows, 256 columns, a fifth of the
// lines from behind the L2) more waves only wait longer: with 12 instead of 16 they wait 0.42 of their time instead of 0.60, the misses stay the
// same, and the L1 stands still for 0.314 of the time instead of 0.323 (800 -> 787 us).  Segments: 16 waves (see above).  Rows of about 40
// entries and more: 12 (besides, 4 M, 50 000 rows, 128 columns 92.9 -> 92.3; 15.3 M, 223 000 rows, 320 columns, the step 935 -> 899), but all that
// fit where rows are shorter, where there are pieces for a turn or two only and for one line per slice (0.83).  81 steps of 6 to 130 entries per
// row, 64 to 600 columns, slices of two and four lines, with 16 and with 12 waves: where the rule takes 12 they are 0.999 to 1.037 times as fast,
// elsewhere 0.91 to 1.04 (above 1.015 in four).
//
// Packed rows, whose workgroups have 52 KB: 8 instead of 12 in slices of four lines with 9 000 waves and 2.2 M entries, or with three lines and
// 18 000 waves.  169 steps of 8 to 150 entries per row, 64 to 600 columns: where the rule takes 8 waves 0.98 to 1.045 times as fast, 1.016 on
// average; with four lines and fewer entries 0.94 to 1.03 (0.987), fewer waves 0.89 to 1.04 (0.976), with three lines and fewer waves 0.80 to
// 1.06 (0.957), with two lines 0.87 to 0.98.
unsigned idle_lds(const adaqp_spmm_pieces *p, const PieceArgs &a, int32_t per_slice, bool packed)
{
    if (p->entries != kEntries || per_slice == 1) return 0;
    const int64_t waves = (int64_t)a.n_pieces * ((a.lines + per_slice - 1) / per_slice);
    if (packed) {
        const bool many = a.lines == 3 ? waves >= 18000 : a.lines > 3 && waves >= 9000 && a.n_walked >= 2200000;
        return per_slice == 4 && many ? kIdleLdsPacked : 0;
    }
    const bool turns = waves >= 9000 || (per_slice == 4 && a.n_walked >= 550 * (int64_t)a.n_pieces);
    return kIdleLds[a.of_rows && turns && a.n_walked >= 40 * (int64_t)a.n_seg];
}

}  // namespace

int launch_pieces(const adaqp_spmm_pieces *p, PieceArgs a, hipStream_t st)
{
    a.pieces = p->pieces_dev;
    a.dest = p->dest_dev;
    a.n_pieces = (int32_t)p->n_pieces;
    a.n_partials = (int32_t)p->n_partials;
    a.ldp = ((int64_t)a.dim + kLine - 1) / kLine * kLine;
    a.n_blocks = (a.n_pieces + p->waves - 1) / p->waves;
    const bool packed = a.p.row != nullptr;
    const int64_t lines = a.ldp / kLine;
    const int32_t per_slice = packed ? packed_lines(p, a, lines) : p->lines_per_slice;
    const int64_t most_lines = pieces_lines(a.n_blocks, p->waves, per_slice);
    for (int64_t l0 = 0; l0 < lines; l0 += most_lines) {
        PieceArgs s = a;
        s.lines = (int32_t)std::min(lines - l0, most_lines);
        s.dim = (int32_t)std::min<int64_t>(a.dim - l0 * kLine, (int64_t)s.lines * kLine);
        s.wdim = s.lines * kLine;
        s.H += l0 * kLine;
        s.p.col0 = (int32_t)(l0 * kLine);
        s.p.full_dim = a.dim;
        s.out += l0 * kLine;
        if (s.partial) s.partial += l0 * kLine;
        s.copy_blocks = packed && l0 == 0 ? (s.copies.blocks() + kXcds - 1) / kXcds * kXcds : 0;
        const dim3 grid((unsigned)(SliceTasks(s.lines, per_slice, s.n_blocks, packed).most_per_xcd() * kXcds) + s.copy_blocks);
        const PieceKernel kernel = packed ? kernel_of<true, true>(p, per_slice) : a.of_rows ? kernel_of<false, true>(p, per_slice) : kernel_of<false, false>(p, per_slice);
        hipLaunchKernelGGL(kernel, grid, dim3(p->waves * kWave), idle_lds(p, s, per_slice, packed), st, s);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    constexpr int64_t kMostSums = (int64_t)1 << 24;         // of a launch, which has fewer than 2^32 threads
    for (int64_t s0 = 0; s0 < p->n_sums; s0 += kMostSums) {
        const int64_t n = std::min(p->n_sums - s0, kMostSums);
        const dim3 grid((unsigned)((n + kWavesPerBlock - 1) / kWavesPerBlock), (unsigned)std::min<int64_t>((a.ldp + kWave * 4 - 1) / (kWave * 4), 64));
        hipLaunchKernelGGL(pieces_sum_kernel, grid, dim3(kBlock), 0, st, p->sum_row_dev + s0,
                           p->sum_ptr_dev + s0, n, a.n_partials, a.partial, a.dim, a.ldp, a.out, a.ldo, a.n_rows);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    return ADAQP_OK;
}

}  // namespace adaqp

using namespace adaqp;

namespace {

// Sums of the `held[q]` largest values, held descending: counted by value below kFew, the few others sorted (1.8 M entries, 269 000 columns: the
// whole rule 6.6 ms, 8.9 with a partial sort per sum).
constexpr int32_t kFew = 4096;

template <int N>
void sums_of_largest(const std::vector<int32_t> &values, const int64_t (&held)[N], int64_t (&sums)[N])
{
    std::vector<int64_t> n_of((size_t)kFew, 0);
    std::vector<int32_t> many;
    int32_t most = 0;                           // of the few
    for (const int32_t v : values) {
        if (v < kFew) {
            ++n_of[(size_t)v];
            most = std::max(most, v);
        } else many.push_back(v);
    }
    std::sort(many.begin(), many.end(), std::greater<int32_t>());
    for (int q = 0; q < N; ++q) {
        const int64_t of_many = std::min<int64_t>(held[q], (int64_t)many.size());
        sums[q] = std::accumulate(many.begin(), many.begin() + of_many, (int64_t)0);
        int64_t left = held[q] - of_many;
        for (int32_t v = most; v > 0 && left > 0; --v) {
            const int64_t n = std::min(left, n_of[(size_t)v]);
            sums[q] += n * v;
            left -= n;
        }
    }
}

}  // namespace

// What lines per slice weigh.  An XCD misses the lines of the columns that its L2 does not hold (32 768 of one line each, the most popular
// ones), which takes 2.4 times as long as a line that it holds; beside that, each slice walks all entries and ends all rows, and a
// narrower last slice leaves lines unused; the two overlap in part.  A launch that does not fill the GPU gains from more slices.
// Weights fitted to 2 890 layer steps of 2 000 to 306 000 rows, 4 to 500 entries per row, 16 to 602 columns of H, Zipf and
// log-normal rows, both directions, one to four lines each.  Geometric mean against shares cut on the device 1.148 (the best lines each
// time 1.166); 2.6 % of the steps are more than 3 % slower, most of them backward steps of 3 to 5 entries per row and many lines, which
// therefore are left as they were (there 0.98 on average).  150 000 x 200 000, 40 entries per row, 256 columns, backward, log-normal
// rows: 1 line 0.89 ms, 4 lines 1.12; Zipf rows, whose columns are few popular ones, 128 columns: 0.27, 0.23.
//
// Segments save what their rows miss; they cost a partial row per group of tiles, written and read, a second copy of the short walk,
// and two more launches.  Where all columns fit, they still are the better ones for long rows: what adaqp_spmm_segments_gain weighs
// counts as well (with the columns that an L2 holds eight lines of as the popular ones).  400 of these steps, timed without blocks as
// well: 1.175 against shares without segments, pieces over the rows alone 1.134, by that gain alone 1.158; 3 with segments lose more
// than 4 % by them, 6 without would gain that.  179 000 rows, 2 M entries, 300 columns: 378 -> 356 us.
extern "C" int adaqp_spmm_pieces_rule(const int64_t *rowptr_host, const int32_t *col_host, int64_t row_begin, int64_t row_end, int64_t n_cols,
                                      int32_t dim, int32_t transposed, int32_t *lines_out, double *segments_gain_out)
{
    if (!rowptr_host || !lines_out || row_begin < 0 || row_end < row_begin || n_cols < 0 || n_cols > INT32_MAX || dim <= 0)
        return ADAQP_EINVAL;
    constexpr int64_t kL2Lines = 32768;         // 4 MB
    constexpr int64_t kSample = 1 << 22;        // entries looked at for the popularity of the columns
    const int64_t first = rowptr_host[row_begin], last = rowptr_host[row_end], block_row = adaqp_spmm_blocks_min_row(n_cols);
    if (first < 0 || last < first || (last > first && !col_host)) return ADAQP_EINVAL;
    const double lines = (double)(((int64_t)dim + 31) / 32), entries = (double)(last - first), rows = (double)(row_end - row_begin);
    double cut = 0.0, n_cut = 0.0, dense = 0.0;
    int64_t n_dense = 0;
    bool ascending = segments_gain_out != nullptr;          // (nobody asks: not looked at)
    for (int64_t r = row_begin; r < row_end; ++r) {
        const int64_t degree = rowptr_host[r + 1] - rowptr_host[r];
        if (degree < 0) return ADAQP_EINVAL;
        if (degree >= ADAQP_SPMM_TILED_SHORT_ROW) {
            cut += (double)degree;
            n_cut += 1.0;
        }
        if (degree >= block_row) {
            dense += (double)degree;
            ++n_dense;
        }
        int32_t before = -1;
        for (int64_t j = rowptr_host[r]; ascending && j < rowptr_host[r + 1]; ++j) {
            ascending = col_host[j] > before && col_host[j] < n_cols;
            before = col_host[j];
        }
    }
    *lines_out = 2;
    if (segments_gain_out) *segments_gain_out = -INFINITY;
    if (segments_gain_out && !ascending && adaqp_spmm_tiled_pays(row_end - row_begin, last - first)) return ADAQP_EINVAL;
    if (last == first) return ADAQP_OK;
    const int64_t stride = std::max<int64_t>((last - first) / kSample, 1), held[4] = {kL2Lines, kL2Lines / 2, kL2Lines / 4, kL2Lines / 8};
    int64_t seen = 0, found[4];                 // entries, and those of the most popular columns
    try {
        std::vector<int32_t> uses((size_t)n_cols, 0);
        for (int64_t j = first; j < last; j += stride)
            if ((uint32_t)col_host[j] < (uint32_t)n_cols) {
                ++uses[(size_t)col_host[j]];
                ++seen;
            }
        sums_of_largest(uses, held, found);
    } catch (const std::bad_alloc &) {          // nothing may be thrown through a C entry; the plan would have no room either
        return ADAQP_OK;
    }
    if (seen == 0) return ADAQP_OK;
    double best = 0.0, missed = 0.0, unpopular = 0.0;
    for (int32_t v = 1, q = 0; v <= 8; v *= 2, ++q) {
        const double miss = 1.0 - (double)found[q] / (double)seen;
        if (v == 8) unpopular = miss;
        const double slices = std::ceil(lines / v), misses = 2.4 * entries * lines * miss, path = (entries + 8.0 * rows) * slices;
        const double held_lines = entries * lines + slices * (0.2 * entries + 2.5 * rows) + 0.4 * (slices * v - lines) * entries;
        const double cost = std::sqrt(misses * misses + held_lines * held_lines) + 2e4 * std::max(0.0, std::log2(1.2e6 / path));
        if (v == 8 || (v > 1 && cost >= best)) continue;
        best = cost;
        missed = miss;
        *lines_out = v;
    }
    if (transposed && entries >= 1e5 && entries < 6.0 * rows && lines >= 7.0) *lines_out = 0;
    if (!ascending) return ADAQP_OK;
    const double groups = (double)std::min<int64_t>(std::max<int64_t>(n_cols / 12288, 1), ADAQP_SPMM_SEGMENTS);
    if (transposed || !adaqp_spmm_blocks_pay(n_dense, n_cols, 32)) dense = 0.0;
    const double by_misses = cut * lines * missed - 7.0 * n_cut * lines * groups - 0.15 * entries - 1e6;
    const double by_popularity = cut * lines * unpopular - segments_cost(transposed != 0, lines, entries, rows) - ADAQP_SPMM_SEGMENTS_MIN_GAIN / 2;
    *segments_gain_out = std::max(by_misses, blocks_gain(lines, dense) + by_popularity);
    return ADAQP_OK;
}

extern "C" int adaqp_spmm_pieces_workspace_bytes(int64_t n_partials, int32_t dim, int64_t *bytes_out)
{
    if (!bytes_out || n_partials < 0 || dim <= 0) return ADAQP_EINVAL;
    if (n_partials > INT32_MAX - 1024) return ADAQP_ESIZE;
    const int64_t wdim = ((int64_t)dim + kLine - 1) / kLine * kLine;
    *bytes_out = (n_partials * wdim * 4 + 255) / 256 * 256;
    return ADAQP_OK;
}

extern "C" int adaqp_plan_spmm_pieces(const int64_t *ptr_host, int64_t n_seg, const int32_t *of_row_host, int64_t n_rows, int32_t dim,
                                      int32_t lines_per_slice, int64_t *sizes_inout, adaqp_spmm_piece *pieces_out, int32_t *dest_out,
                                      int32_t *sum_row_out, int32_t *sum_ptr_out)
try {
    constexpr int S = ADAQP_SPMM_SEGMENTS;
    if (n_seg < 0 || n_rows < 0 || dim <= 0 || !ptr_host || !sizes_inout || ptr_host[0] < 0 || (!of_row_host && n_rows != n_seg)) return ADAQP_EINVAL;
    if (lines_per_slice != 1 && lines_per_slice != 2 && lines_per_slice != 4) return ADAQP_EINVAL;
    if (n_seg > INT32_MAX - 1024 || n_rows > INT32_MAX - 1024) return ADAQP_ESIZE;
    const bool fill = pieces_out != nullptr;
    if (fill && ((n_seg > 0 && !dest_out) || !sum_ptr_out || (sizes_inout[2] > 0 && !sum_row_out))) return ADAQP_EINVAL;
    for (int64_t s = 0; s < n_seg; ++s)
        if (ptr_host[s + 1] < ptr_host[s]) return ADAQP_EINVAL;
    const PieceShape shape = piece_shape(n_seg, ptr_host[n_seg] - ptr_host[0], dim, lines_per_slice);

    // Pieces of whole segments; one that would be less than half full takes the next segment up to a line of entries.  In the large
    // workgroups the parts of a segment are one workgroup's wherever they can be: pieces of nothing before them.
    std::vector<adaqp_spmm_piece> pieces{{ptr_host[0], 0, -1}};
    std::vector<int32_t> cuts((size_t)n_seg, 0);            // of a segment, but for joined ones
    int64_t looked_at = -1;                                 // the last segment that was cut, and whether its parts are joined
    bool joins = false;
    for (int64_t seg = 0, entry = ptr_host[0]; seg < n_seg;) {
        const int64_t first_seg = seg, first = entry;
        auto weight = [&](int64_t e, int64_t s) { return e - first + 8 * (s - first_seg); };
        while (seg < n_seg && seg - first_seg < kEnds && ptr_host[seg + 1] - first <= shape.entries && weight(ptr_host[seg + 1], seg + 1) <= shape.length)
            entry = ptr_host[++seg];
        int32_t partial = -1;
        if (seg < n_seg && seg - first_seg < kEnds && weight(entry, seg) < shape.length / 2) {
            auto cut_at = [&](int64_t from, int64_t ends) { return (from + std::min<int64_t>(shape.length - 8 * ends, shape.entries)) / 32 * 32; };
            const int64_t to = cut_at(first, seg - first_seg), end = ptr_host[seg + 1];
            if (to > entry && to < end) {
                const int64_t in_group = (int64_t)(pieces.size() - 1) % shape.waves;
                if (shape.waves == kJoinWaves && looked_at != seg) {        // its first part: how many there will be
                    int64_t parts = 2;
                    for (int64_t e = to, next; parts <= shape.waves && (next = cut_at(e, 0)) < end && end - e + 8 > shape.length; e = next) ++parts;
                    joins = parts <= shape.waves;
                    if (joins && in_group + parts > shape.waves) {
                        if (entry > first || seg > first_seg) pieces.push_back({entry, (int32_t)seg, -1});
                        while ((pieces.size() - 1) % shape.waves) pieces.push_back({entry, (int32_t)seg, -1});
                        continue;
                    }
                }
                looked_at = seg;
                entry = to;
                partial = joins ? kJoined : cuts[(size_t)seg]++;
            }
        }
        if (entry == first && seg == first_seg) entry = ptr_host[++seg];        // a segment a little over the length
        pieces.push_back({entry, (int32_t)seg, partial});
        if ((int64_t)pieces.size() > kMostPieces) return ADAQP_ESIZE;
    }

    // A row of one segment that is not cut is written at once; the others' partial rows lie in the order of the rows.
    std::vector<int32_t> dest((size_t)n_seg, INT32_MIN), sum_row, sum_ptr{0};
    int64_t n_partials = 0;
    for (int64_t r = 0; r < n_rows; ++r) {
        const int32_t row_itself[S] = {(int32_t)r, -1, -1, -1, -1, -1, -1, -1}, *of = of_row_host ? of_row_host + r * S : row_itself;
        if (of[0] < -1) continue;                           // someone else's
        int parts = 0;
        int32_t only = -1;
        for (int q = 0; q < S; ++q) {
            if (of[q] < 0) continue;
            if (of[q] >= n_seg || dest[(size_t)of[q]] != INT32_MIN) return ADAQP_EINVAL;
            parts += 1 + cuts[(size_t)of[q]];
            only = of[q];
            dest[(size_t)only] = 0;
        }
        if (parts == 1) {
            dest[(size_t)only] = (int32_t)(-1 - r);
            continue;
        }
        for (int q = 0; q < S; ++q) {
            if (of[q] < 0) continue;
            n_partials += cuts[(size_t)of[q]];
            if (n_partials > INT32_MAX - 1024) return ADAQP_ESIZE;
            dest[(size_t)of[q]] = (int32_t)n_partials++;
        }
        sum_row.push_back((int32_t)r);
        sum_ptr.push_back((int32_t)n_partials);
    }
    for (int64_t s = 0; s < n_seg; ++s)
        if (dest[(size_t)s] == INT32_MIN) return ADAQP_EINVAL;
    for (size_t p = 1; p < pieces.size(); ++p)
        if (pieces[p].partial >= 0) {
            const size_t s = (size_t)pieces[p].segment;
            pieces[p].partial += dest[s] - cuts[s];
        }
    const int64_t sizes[5] = {(int64_t)pieces.size() - 1, n_partials, (int64_t)sum_row.size(), shape.waves, shape.entries};
    if (!fill) {
        std::copy(sizes, sizes + 5, sizes_inout);
        return ADAQP_OK;
    }
    if (!std::equal(sizes, sizes + 5, sizes_inout)) return ADAQP_EINVAL;
    std::copy(pieces.begin(), pieces.end(), pieces_out);
    std::copy(dest.begin(), dest.end(), dest_out);
    std::copy(sum_row.begin(), sum_row.end(), sum_row_out);
    std::copy(sum_ptr.begin(), sum_ptr.end(), sum_ptr_out);
    return ADAQP_OK;
} catch (const std::bad_alloc &) {           // nothing may be thrown through a C entry
    return ADAQP_ESIZE;
}
