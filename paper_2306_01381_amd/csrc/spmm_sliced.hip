// Neighbour aggregation (Sec. 2.1 Eq. 3) with the feature columns sliced over the XCDs.  Made for the line-padded layout;
// takes rows that start anywhere too.
//
// The gather is bound by what comes from behind the L2s: rows of H are drawn from a power law with no locality, every
// XCD has a private 4 MB L2, and when all eight walk whole rows (1 KB and more) each holds the same few thousand
// popular rows.  Here an XCD walks the graph for ITS share of the feature columns only, a slice of VPL 128-byte lines
// of every row at a time: its L2 then holds one line of 32 768 rows (four of 8 192) instead of eight or more lines of
// 4 000, the L2s hold different data, and no line of H is fetched behind two of them.  The price is that the entries
// (8 bytes each) are read once per slice.
//
// Work split: a wave walks a contiguous share of the merge path of row ends and entries (as in spmm.hip).  Its entries
// go through LDS 8 at a time: one load instruction per line fetches the lines of 8 consecutive entries, a lane holding
// four columns of one of them, and kAhead such steps are in flight at any time, across row ends and across the chunks
// in which entries are staged.  A step in which no row ends costs one LDS read, one add and 4 multiply-adds per line;
// where a row ends, the products of the groups before the end are added to the row's sums, these are added across the
// eight groups (halving the registers at each level) and stored, and the products after it start the next row.  The row
// a share begins in is finished by the carry kernel, from the part that the share before it left.  The summation
// order depends on the launch geometry only.
//
// Bound: what a slice misses in its L2 (306 000 x 456 000, 256 columns: 17 % hits, 7.3 TB/s behind the L2s), and where it fits,
// the rate at which a CU takes 16-byte gathers (32 TB/s over the chip for bare loads out of L2; this loop 25-28, and 19.8 with
// 81 % hits on the transposed graph below).  Measured against the merge-path kernel
// walking whole rows (aggregation of all rows, before -> after): 50 000 x 30 000, 4 M entries, 128 columns 0.239 ->
// 0.096 ms; 34 000 columns, 0.42 M entries, 66 columns 0.050 -> 0.027; 376 000 x 196 000, 16.2 M entries, 256 columns
// (transposed graph) 0.96 -> 0.80; 306 000 x 456 000, 7.7 M entries, 256 columns 1.13 -> 1.07; 179 000 x 269 000, 2 M
// entries, 300 columns 0.386 -> 0.361.  Packed rows cost a slot lookup per entry and slice and fetch whole lines of codes for a
// part of them: 66 columns 1.6-2.7 times as fast as the merge path, 256 columns 1.1-1.5, 400 to 602 columns 0.83-1.2.  Tried on the way: a piece of the path per group of eight lanes (every row end
// then stops seven other rows), steps padded to row ends (a third of the gather slots fetch nothing), and repeating an
// entry in idle slots instead of an offset outside the buffer (the L1 stalls on a line that is already on its way).
#include <algorithm>

#include "spmm_common.hpp"

namespace adaqp {
namespace {

constexpr int64_t kMinPath = 1024;                  // of a workgroup's four shares
constexpr int kStep = 8;                            // entries of a step = groups of a wave
constexpr int kGroup = kWave / kStep;               // lanes per entry: 8 x 16 bytes = one line
constexpr int kLine = 32;                           // columns per line
constexpr int kPer = 6;                             // entries a lane stages per chunk
constexpr int kChunk = kPer * kWave;                // entries of a chunk: a whole number of rings for every VPL
constexpr int kEnds = kWave - 1;                    // row ends of a chunk at most
constexpr int32_t kNoEnd = 0x10000;                 // lies after every step of a chunk
constexpr int kRowSteps = 8;                        // entries a row end counts for where shares are cut
constexpr int kNonTemporal = 2;                     // cache policy bits of a buffer load: nt
constexpr int kRawBuffer = 0x00020000;              // buffer resource, last word: raw 32-bit data, no swizzle

struct SlicedArgs {
    SpmmArgs s;
    int32_t n_blocks;           // workgroups per slice, kWavesPerBlock shares each
    int32_t lines;              // lines of a row
};

typedef float float4_t __attribute__((ext_vector_type(4)));

// An entry in LDS: byte offset of its row of H and its coefficient.  PACKED: bits 0-1 of the offset name the width of
// a row that is still packed (1, 2, 3: 2, 4, 8 bits; the offset is then one into the receive buffer) and (Z, S) follow.
template <bool PACKED> struct Entry;
template <> struct alignas(8) Entry<false> { uint32_t off; float val; };
template <> struct alignas(16) Entry<true> { uint32_t off; float val; float z, s; };

template <int U, int N, typename F>
__device__ __forceinline__ void unroll(F &&f)
{
    if constexpr (U < N) {
        f(std::integral_constant<int, U>());
        unroll<U + 1, N>(f);
    }
}

// Row ends before two diagonals of the merge path: row end p precedes d iff end_p + kRowSteps * (p + 1) <= d.  256-ary
// search by a whole wave; wave-uniform results.
__device__ void split_rows2(const SpmmArgs &a, const int64_t (&d)[2], int64_t base, int64_t nnz_r, int lane, int32_t (&at)[2])
{
    constexpr int K = kProbes / kWave;
    int32_t lo[2], hi[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int64_t least = d[q] - nnz_r > 0 ? (d[q] - nnz_r) / kRowSteps : 0, most = d[q] / kRowSteps;
        hi[q] = (int32_t)(most < a.n_rows ? most : a.n_rows);
        lo[q] = (int32_t)(least < hi[q] ? least : hi[q]);
    }
    while (lo[0] < hi[0] || lo[1] < hi[1]) {
        bool before[2][K];
        int32_t step[2], probes[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int32_t n = hi[q] - lo[q];
            step[q] = (n + K * kWave - 1) / (K * kWave);
            probes[q] = n > 0 ? (n + step[q] - 1) / step[q] : 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int32_t i = k * kWave + lane;
                before[q][k] = false;
                if (i < probes[q]) {
                    const int64_t p = (int64_t)lo[q] + (int64_t)i * step[q];
                    before[q][k] = clamp64(a.rowptr[p + 1], base, base + nnz_r) - base + kRowSteps * (p + 1) <= d[q];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int32_t cnt = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) cnt += __popcll(__ballot(before[q][k]));
            const int32_t new_lo = cnt > 0 ? lo[q] + (cnt - 1) * step[q] + 1 : lo[q];
            const int32_t new_hi = cnt < probes[q] ? lo[q] + cnt * step[q] : hi[q];
            lo[q] = new_lo;
            hi[q] = new_hi;
        }
    }
    at[0] = __builtin_amdgcn_readfirstlane(lo[0]);
    at[1] = __builtin_amdgcn_readfirstlane(lo[1]);
}

// x and y hold two values per lane for two halves of the wave (HALF = 32) or of each half (16): afterwards a lane of the
// lower half holds the sum of both halves' x, a lane of the upper half that of both halves' y.
template <int HALF>
__device__ __forceinline__ float fold(float x, float y)
{
    typedef unsigned pair_t __attribute__((ext_vector_type(2)));
    const uint32_t ux = __builtin_bit_cast(uint32_t, x), uy = __builtin_bit_cast(uint32_t, y);
    pair_t r;
    if constexpr (HALF == 32) r = __builtin_bit_cast(pair_t, __builtin_amdgcn_permlane32_swap(ux, uy, false, false));
    else                      r = __builtin_bit_cast(pair_t, __builtin_amdgcn_permlane16_swap(ux, uy, false, false));
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

__device__ __forceinline__ float ror8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int32_t, v), 0x128, 0xF, 0xF, false));
}

// One wave's share of the path for one slice of VPL lines.  WHOLE: rows of H and out start on lines and have whole lines
// of room.  Otherwise rows start anywhere (4-byte aligned) and end after a.dim columns: a lane whose four columns would
// not end in the row takes the row's last four, and columns that two lanes hold are stored twice with the same bits.
template <int VPL, bool PACKED, bool WHOLE>
__device__ void walk_share(const SlicedArgs &sa, const int32_t first_line, const int32_t item, Entry<PACKED> (*stages)[kChunk])
{
    constexpr int kAhead = VPL >= 3 ? 2 : 8 / VPL;          // steps in flight: 6 to 8 KB per wave
    constexpr int kRing = kAhead * kStep;                   // entries of a turn of the ring
    static_assert(kChunk % kRing == 0, "a chunk is a whole number of turns");
    const SpmmArgs &a = sa.s;
    const int lane = threadIdx.x & (kWave - 1), gl = lane & (kGroup - 1), grp = lane / kGroup;

    // extent of the range on the device: the host only sized the launch
    const int64_t base = clamp64(a.rowptr[0], 0, a.nnz);
    const int64_t nnz_r = clamp64(a.rowptr[a.n_rows], base, a.nnz) - base;
    const int64_t total = (int64_t)a.n_rows * kRowSteps + nnz_r;
    const int64_t n_items = (int64_t)sa.n_blocks * kWavesPerBlock;
    const int64_t per = (total + n_items - 1) / n_items;
    int64_t d[2];
    d[0] = item * per < total ? item * per : total;
    d[1] = d[0] + per < total ? d[0] + per : total;
    int32_t i[2];
    split_rows2(a, d, base, nnz_r, lane, i);
    int64_t j[2];                                           // entries before a diagonal: those of the open row up to it,
#pragma unroll                                              // none of the weight of its end
    for (int q = 0; q < 2; ++q) {
        const int64_t end = i[q] < a.n_rows ? clamp64(a.rowptr[(int64_t)i[q] + 1], base, base + nnz_r) - base : nnz_r;
        j[q] = clamp64(d[q] - (int64_t)kRowSteps * i[q], 0, end);
    }
    if (j[1] < j[0]) j[1] = j[0];

    const int32_t c0 = first_line * kLine + gl * 4;         // first column of the lane's line 0
    // one buffer per line of the slice; rows of any length: one buffer, and the lane's column in each line
    __amdgpu_buffer_rsrc_t rows[VPL];
    uint32_t lane_off[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int32_t begin = WHOLE ? (first_line + v) * kLine : 0;
        rows[v] = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.H + begin), 0,
                                                    (int)(uint32_t)(a.n_cols * a.ldh * 4 - begin * 4), kRawBuffer);
        lane_off[v] = WHOLE ? gl * 16 : (uint32_t)min(c0 + v * kLine, a.dim - 4) * 4;
    }
    const auto packed_rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.packed), 0,
                                                               (int)(uint32_t)a.packed_bytes, kRawBuffer);
    const uint32_t pitch = (uint32_t)a.ldh * 4u;

    // After `sum_groups` lane l (and lane l + 32) holds column l of each line.
    const int line_col = lane & (kLine - 1);
    const int from_lane = ((line_col & 3) * 16 + line_col / 4) << 2;
    auto column_of = [&](int v) {                           // the column lane l holds a sum of; negative: none of its own
        const int32_t line = (first_line + v) * kLine;
        if constexpr (WHOLE) return line + line_col;
        const int32_t four = line + (line_col & ~3);
        return four < a.dim ? min(four, a.dim - 4) + (line_col & 3) : -1;
    };
    auto sum_groups = [&](const float4_t (&acc)[VPL], float (&out)[VPL]) {
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const float lo = fold<32>(acc[v][0], acc[v][2]), hi = fold<32>(acc[v][1], acc[v][3]);
            float x = fold<16>(lo, hi);                     // row q of 16 lanes: column 4 * gl + q, twice
            x = x + ror8(x);
            out[v] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from_lane, __builtin_bit_cast(int32_t, x)));
        }
    };

    // The share is walked in chunks of up to kChunk entries and kEnds row ends.  What a chunk needs from memory is
    // requested one chunk ahead and waits in registers: bounds of rows, one per lane, and entries.
    struct Chunk {
        int32_t row0, n_end, n_ent;                         // first row, row ends, entries
        int64_t ent0;                                       // first entry
        int32_t ends;                                       // lane l: where row row0 + l ends in the chunk, else kNoEnd
    };
    int64_t r_hi;
    auto request_rows = [&](int32_t row) {
        const int64_t r = (int64_t)row + lane + 1;
        r_hi = a.rowptr[r < a.n_rows ? r : a.n_rows];
    };
    auto take = [&](int32_t row0, int64_t ent0) {           // from r_hi, requested for row0
        Chunk c;
        c.row0 = row0;
        c.ent0 = ent0;
        const int64_t end = clamp64(clamp64(r_hi, base, base + nnz_r) - base - ent0, 0, kNoEnd);
        c.ends = (int32_t)end;
        const int64_t left = j[1] - ent0;
        c.n_ent = (int32_t)(left < kChunk ? left : kChunk);
        c.n_end = __popcll(__ballot(lane < kEnds && row0 + lane < i[1] && c.ends <= c.n_ent));
        if (c.n_end == kEnds) c.n_ent = min(c.n_ent, __builtin_amdgcn_readlane(c.ends, kEnds - 1));
        if (lane >= c.n_end) c.ends = kNoEnd;
        return c;
    };
    int32_t st_col[kPer];
    float st_val[kPer];
    auto request_entries = [&](const Chunk &c) {            // past the chunk's entries: zeros
        const auto cols = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(a.col + base + c.ent0), 0, c.n_ent * 4, kRawBuffer);
        const auto vals = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.val + base + c.ent0), 0, c.n_ent * 4, kRawBuffer);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {                    // streamed: keep the caches for H
            const int at = lane * 4 + k * kWave * 4;        // all of it here: the scalar offset is outside the range check
            st_col[k] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(cols, at, 0, kNonTemporal);
            st_val[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vals, at, 0, kNonTemporal));
        }
    };
    auto stage = [&](const Chunk &c, Entry<PACKED> *ent) {
        Entry<PACKED> en[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int32_t col = st_col[k];
            const bool ok = k * kWave + lane < c.n_ent && col >= 0 && col < a.n_cols;       // else: fetches nothing
            en[k] = {};
            en[k].off = ok ? (uint32_t)col * pitch : kOutside;
            en[k].val = ok ? st_val[k] : 0.0f;
        }
        if constexpr (PACKED) {
            // all lookups of a chunk are on their way together, those of entries without a slot at index 0: behind a branch
            // each they would wait for one another, six times two latencies per chunk
            int32_t slot[kPer], b[kPer];
            int64_t off[kPer];
            float2 zs[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) slot[k] = a.slot_of_row[en[k].off != kOutside ? st_col[k] : 0];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const bool has = en[k].off != kOutside && slot[k] >= 0 && slot[k] < a.n_slots;
                slot[k] = has ? slot[k] : -1;
                const int64_t at = has ? slot[k] : 0;
                b[k] = a.bits[at];
                off[k] = a.row_offset[at];
                zs[k] = *reinterpret_cast<const float2 *>(a.params + 2 * at);
            }
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int64_t stride = 4 * (((int64_t)a.full_dim * b[k] + 31) >> 5);
                if (slot[k] >= 0 && (b[k] == 2 || b[k] == 4 || b[k] == 8) && off[k] >= 0 && (off[k] & 3) == 0 &&
                    off[k] + stride <= a.packed_bytes) {
                    en[k].off = (uint32_t)off[k] | (b[k] == 2 ? 1u : (b[k] == 4 ? 2u : 3u));
                    en[k].z = zs[k].x;
                    en[k].s = zs[k].y;
                }                                           // else: the row in H
            }
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) ent[k * kWave + lane] = en[k];
    };

    // the ring: kAhead steps whose lines are on their way
    float4_t h[kAhead][VPL];
    uint32_t words[kAhead][VPL], words_up[kAhead][VPL];     // four codes, where rows end anywhere across two words
    Entry<PACKED> in_flight[kAhead];
    auto packed_col = [&](int v) { return (uint32_t)a.col0 + (WHOLE ? (uint32_t)(c0 + v * kLine) : lane_off[v] / 4); };
    auto fetch = [&](auto tag, const Entry<PACKED> &en) {
        constexpr int U = decltype(tag)::value;
        in_flight[U] = en;
        const uint32_t w = PACKED ? en.off & 3u : 0u;
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const uint32_t off = PACKED && w != 0 ? kOutside : en.off + lane_off[v];
            h[U][v] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(rows[v], (int)off, 0, 0));
            if constexpr (PACKED) {
                // one 32-bit word holds the four codes of a lane whose first column is a multiple of four (4 * b <= 32 and
                // divides 32)
                const uint32_t last_word = (((uint32_t)a.full_dim << w) - 1) >> 5;
                const uint32_t word = (packed_col(v) << w) >> 5;
                words[U][v] = __builtin_amdgcn_raw_buffer_load_b32(
                    packed_rows, w != 0 ? (int)((en.off & ~3u) + 4 * min(word, last_word)) : (int)kOutside, 0, 0);
                if constexpr (!WHOLE)
                    words_up[U][v] = __builtin_amdgcn_raw_buffer_load_b32(
                        packed_rows, w != 0 ? (int)((en.off & ~3u) + 4 * min(word + 1, last_word)) : (int)kOutside, 0, 0);
            }
        }
    };
    auto neighbour = [&](auto tag, int v) {                 // the four columns a lane fetched
        constexpr int U = decltype(tag)::value;
        float4_t x = h[U][v];
        if constexpr (PACKED) {
            const uint32_t w = in_flight[U].off & 3u;
            if (w != 0) {
                const uint32_t b = 1u << w, shift = (packed_col(v) << w) & 31u;
                uint32_t word = words[U][v] >> shift;
                if constexpr (!WHOLE) word = (uint32_t)(((uint64_t)words_up[U][v] << 32 | words[U][v]) >> shift);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float scaled = (float)__builtin_amdgcn_ubfe(word, k * b, b) * in_flight[U].s; // Eq. 5: product
                    x[k] = scaled + in_flight[U].z;                                             // rounded, then sum rounded
                }
            }
        }
        return x;
    };

    // Sums of the open row: acc what the present chunk has given so far, per group; before what earlier chunks of the share
    // gave, as `sum_groups` leaves it.  No addition chain is longer than a chunk's 48 steps, the chunks of a share, or the
    // shares of a row (one running sum over a share would be thousands of terms long and rounds accordingly).
    float4_t acc[VPL];
    float before[VPL];
    bool has_before = false;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        before[v] = 0.0f;
    }
    auto take_sums = [&](float (&sum)[VPL]) {               // and start anew
        sum_groups(acc, sum);
        if (has_before) {
#pragma unroll
            for (int v = 0; v < VPL; ++v) sum[v] = before[v] + sum[v];
            has_before = false;
        }
#pragma unroll
        for (int v = 0; v < VPL; ++v) acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
    };
    float *out_row = a.out + (int64_t)i[0] * a.ldo;         // the rows of a share end one after the other
    auto finish_row = [&]() {
        float sum[VPL];
        take_sums(sum);
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const int32_t c = column_of(v);
            if constexpr (WHOLE) {
                if (lane < kLine) __builtin_nontemporal_store(c < a.dim ? sum[v] : 0.0f, out_row + (uint32_t)c);
            } else {                                        // lines are shared with other rows: left for the L2 to merge
                if (lane < kLine && c >= 0) out_row[c] = sum[v];
            }
        }
        out_row += a.ldo;
    };

    request_rows(i[0]);
    Chunk cur = take(i[0], j[0]);
    request_entries(cur);
    request_rows(cur.row0 + cur.n_end);
    int buf = 0;
    stage(cur, stages[0]);
    unroll<0, kAhead>([&](auto tag) {
        fetch(tag, stages[0][decltype(tag)::value * kStep + grp]);
        __builtin_amdgcn_sched_barrier(0);                  // the order of issue is the order of use
    });
    for (;;) {
        const int32_t next_row = cur.row0 + cur.n_end;
        const int64_t next_ent = cur.ent0 + cur.n_ent;
        Chunk next = take(next_row, next_ent);
        const bool more = next.n_end > 0 || next.n_ent > 0;
        if (more) {
            request_entries(next);
            request_rows(next.row0 + next.n_end);
        }
        int32_t e = 0, end = __builtin_amdgcn_readlane(cur.ends, 0);       // next row end
        while (end == 0) {                                  // ends that belong to what the chunks before have added up
            finish_row();
            end = __builtin_amdgcn_readlane(cur.ends, ++e);
        }
        const int32_t turns = cur.n_ent > 0 ? (cur.n_ent + kRing - 1) / kRing : 1;
        for (int32_t t = 0; t < turns; ++t) {
            const Entry<PACKED> *src = stages[buf] + (t + 1) * kRing + grp;
            if (t + 1 == turns) {                           // the ring goes on in the next chunk
                if (more) stage(next, stages[buf ^ 1]);
                else if (lane < kRing) stages[buf ^ 1][lane] = Entry<PACKED>{kOutside, 0.0f};
                src = stages[buf ^ 1] + grp;
            }
            Entry<PACKED> en = src[0];
            unroll<0, kAhead>([&](auto tag) {
                constexpr int U = decltype(tag)::value;
                const Entry<PACKED> now = en;
                if (U + 1 < kAhead) en = src[(U + 1) * kStep];
                __builtin_amdgcn_sched_barrier(0);
                const int32_t rel = end - t * kRing - U * kStep;        // where in this step a row ends
                float4_t unpacked[VPL];                         // once per step; plain rows as they came
                if constexpr (PACKED) {
#pragma unroll
                    for (int v = 0; v < VPL; ++v) unpacked[v] = neighbour(tag, v);
                }
                auto &x = *(PACKED ? &unpacked : &h[U]);
                if (rel > kStep) {
#pragma unroll
                    for (int v = 0; v < VPL; ++v)
#pragma unroll
                        for (int k = 0; k < 4; ++k) acc[v][k] = fmaf(in_flight[U].val, x[v][k], acc[v][k]);
                } else {
                    // the groups from the last end to this one belong to the row that ends here
                    int32_t from = 0, to = rel;
                    do {
                        const bool mine = grp >= from && grp < to;
#pragma unroll
                        for (int v = 0; v < VPL; ++v)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const float sum = fmaf(in_flight[U].val, x[v][k], acc[v][k]);
                                acc[v][k] = mine ? sum : acc[v][k];
                            }
                        finish_row();
                        end = __builtin_amdgcn_readlane(cur.ends, ++e);
                        from = to;
                        to = end - t * kRing - U * kStep;
                    } while (to <= kStep);
#pragma unroll
                    for (int v = 0; v < VPL; ++v)
#pragma unroll
                        for (int k = 0; k < 4; ++k) acc[v][k] = grp >= from ? in_flight[U].val * x[v][k] : 0.0f;
                }
                fetch(tag, now);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        if (!more) break;
        float sum[VPL];                                     // the open row goes on in the next chunk
        take_sums(sum);
#pragma unroll
        for (int v = 0; v < VPL; ++v) before[v] = sum[v];
        has_before = true;
        cur = next;
        buf ^= 1;
    }
    // what is left belongs to a row that goes on in the next wave's share
    const int64_t began = i[1] < a.n_rows ? clamp64(a.rowptr[i[1]], base, base + nnz_r) - base : nnz_r;
    const bool held = i[1] < a.n_rows && j[1] > (began > j[0] ? began : j[0]);
    if (held) {
        float sum[VPL];
        take_sums(sum);
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            if (lane < kLine && column_of(v) >= 0) a.carry[(int64_t)item * a.carry_ld + column_of(v)] = sum[v];
    }
    if (first_line == 0 && lane == 0) a.carry_row[item] = held ? i[1] : -1;
}

template <int VPL, bool PACKED, bool WHOLE>
__global__ __launch_bounds__(kBlock, 2) void spmm_sliced_kernel(const SlicedArgs sa)
{
    __shared__ Entry<PACKED> stages[kWavesPerBlock][2][kChunk];
    const SliceTasks tasks(sa.lines, VPL, sa.n_blocks, PACKED);
    const int32_t xcd = blockIdx.x % kXcds;
    const int64_t task = tasks.first_task(xcd) + blockIdx.x / kXcds;
    if (task >= tasks.first_task(xcd + 1)) return;
    const int32_t slice = (int32_t)(task / sa.n_blocks), blk = (int32_t)(task % sa.n_blocks);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t item = blk * kWavesPerBlock + wave;
    const int live = min(VPL, sa.lines - slice * VPL);
    if (live == VPL) walk_share<VPL, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    else if (VPL > 3 && live == 3) walk_share<3, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    else if (VPL > 2 && live == 2) walk_share<2, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    else walk_share<1, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
}

}  // namespace

SlicedCut plan_sliced(const SpmmArgs &a, int64_t nnz_hint, bool whole_lines, bool skewed_columns)
{
    if (!sliced_takes(a.n_rows, a.nnz, a.n_cols, a.ldh, a.slot_of_row != nullptr, a.packed_bytes, a.full_dim)) return {0, 0, 0};
    if (!whole_lines && a.dim < 4) return {0, 0, 0};        // a lane takes four columns
    return sliced_cut(a.n_rows, nnz_hint, a.n_cols, (a.wdim + kLine - 1) / kLine, whole_lines, skewed_columns);
}

hipError_t launch_sliced(const SpmmArgs &a, const SlicedCut &cut, int64_t nnz_hint, bool whole_lines, hipStream_t st,
                         int32_t *n_carries_out)
{
    SlicedArgs sa;
    sa.s = a;
    sa.lines = (a.wdim + kLine - 1) / kLine;
    const int vpl = a.slot_of_row ? cut.packed_lines : cut.lines;
    // each wave takes one share, of at least 256 steps of the path: a search and an empty ring each
    const int64_t path = nnz_hint + (int64_t)a.n_rows * kRowSteps;
    int64_t n_blocks = std::min(cut.n_blocks, (path + kMinPath - 1) / kMinPath);
    if (n_blocks > a.n_items / kWavesPerBlock) n_blocks = a.n_items / kWavesPerBlock;      // one carry slot per share
    if (n_blocks < 1) n_blocks = 1;
    sa.n_blocks = (int32_t)n_blocks;
    const dim3 grid((unsigned)(SliceTasks(sa.lines, vpl, sa.n_blocks, a.slot_of_row != nullptr).most_per_xcd() * kXcds));
#define ADAQP_SLICED(V, WHOLE)                                                                                   \
    do {                                                                                                         \
        if (a.slot_of_row) hipLaunchKernelGGL((spmm_sliced_kernel<V, true, WHOLE>), grid, dim3(kBlock), 0, st, sa); \
        else hipLaunchKernelGGL((spmm_sliced_kernel<V, false, WHOLE>), grid, dim3(kBlock), 0, st, sa);           \
    } while (0)
    if (!whole_lines) ADAQP_SLICED(4, false);
    else if (vpl == 1) ADAQP_SLICED(1, true);
    else if (vpl == 2) ADAQP_SLICED(2, true);
    else ADAQP_SLICED(4, true);
#undef ADAQP_SLICED
    *n_carries_out = sa.n_blocks * kWavesPerBlock;
    return hipGetLastError();
}

}  // namespace adaqp
