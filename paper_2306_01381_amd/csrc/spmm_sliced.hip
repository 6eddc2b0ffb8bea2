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
// go through LDS in chunks: one load instruction per line fetches the lines of 8 consecutive entries, a lane holding
// four columns of one of them, and kAhead such steps are in flight at any time, across row ends and across chunks.
// A step in which no row ends (a bit per step says so) costs half an LDS read, one add, one jump and 4 multiply-adds per
// line; where a row ends, the products of the groups before the end are added to the row's sums, these are added across the
// eight groups (halving the registers at each level) and stored, and the products after it start the next row.  The row
// a share begins in is finished by the carry kernel, from the part that the share before it left.  The summation
// order depends on the launch geometry only.
//
// The L1 answers loads in order: a load of entries, which always comes from behind the L2, holds up every gather of the CU
// that would hit (bare gathers with 3 KB of entries per 48 of them: 21 TB/s where the entries come from memory, 28 where they
// are in the L2; 24-25 if four times as many are asked for four times as rarely).  So chunks are large, a lane loads four
// entries at a time and no line of col or val is asked for twice: chunks begin at multiples of a line once the first is over.
// 8 M entries in rows of 2 048, 20 000 columns, 256 columns of H, one line per slice: 384 entries per chunk and four
// per lane and load apart 18.0 TB/s, so 21.0; 30 000 x 20 000 backward step of 4 M entries 109 -> 106 us.
//
// Bound: what a slice misses in its L2 (306 000 x 456 000, 256 columns: 17 % hits, 7.3 TB/s behind the L2s), and where it fits,
// the rate at which a CU takes 16-byte gathers (32 TB/s over the chip for bare loads out of L2; this loop 25-28, and 19.8 with
// 81 % hits on the transposed graph below).  Columns of H must not all fall on the same channels of an L2: a pitch of 8 lines
// costs a slice of one line a quarter of its rate (28 M entries, 98 000 columns: 2.48 ms, 1.93 at a pitch of 9).  Measured against the merge-path kernel
// walking whole rows (aggregation of all rows, before -> after): 50 000 x 30 000, 4 M entries, 128 columns 0.239 ->
// 0.096 ms; 34 000 columns, 0.42 M entries, 66 columns 0.050 -> 0.027; 376 000 x 196 000, 16.2 M entries, 256 columns
// (transposed graph) 0.96 -> 0.80; 306 000 x 456 000, 7.7 M entries, 256 columns 1.13 -> 1.07; 179 000 x 269 000, 2 M
// entries, 300 columns 0.386 -> 0.361.  Packed rows cost a slot lookup per entry and slice and fetch whole lines of codes for a
// part of them: 66 columns 1.6-2.7 times as fast as the merge path, 256 columns 1.1-1.5, 400 to 602 columns 0.83-1.2.  Tried on the way: a piece of the path per group of eight lanes (every row end
// then stops seven other rows), steps padded to row ends (a third of the gather slots fetch nothing), and repeating an
// entry in idle slots instead of an offset outside the buffer (the L1 stalls on a line that is already on its way).
#include <algorithm>

#include "spmm_common.hpp"
#include "spmm_wave.hpp"

namespace adaqp {
namespace {

constexpr int64_t kMinPath = 1024;                  // of a workgroup's four shares

constexpr int kLoads = 3;                           // of four entries per lane: what a chunk takes of col, and of val
constexpr int kChunk = kLoads * 4 * kWave;          // entries of a chunk
constexpr int kPart = kChunk / 2;                   // no sum runs longer: a whole number of rings for every VPL
constexpr int kEnds = kWave - 1;                    // row ends of a chunk at most
constexpr int32_t kNoEnd = 0x10000;                 // lies after every step of a chunk
constexpr int kRowSteps = 8;                        // entries a row end counts for where shares are cut


struct SlicedArgs {
    SpmmArgs s;
    int32_t n_blocks;           // workgroups per slice, kWavesPerBlock shares each
    int32_t lines;              // lines of a row
};

// Row ends before two diagonals of the merge path: row end p precedes d iff end_p + kRowSteps * (p + 1) <= d.  256-ary
// search by a whole wave; wave-uniform results.
__device__ __forceinline__ void split_rows2(const SpmmArgs &a, const int64_t (&d)[2], int64_t base, int64_t nnz_r, int lane, int32_t (&at)[2])
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

// One wave's share of the path for one slice of VPL lines.  WHOLE: rows of H and out start on lines and have whole lines
// of room.  Otherwise rows start anywhere (4-byte aligned) and end after a.dim columns: a lane whose four columns would
// not end in the row takes the row's last four, and columns that two lanes hold are stored twice with the same bits.
template <int VPL, bool PACKED, bool WHOLE>
__device__ __forceinline__ void walk_share(const SlicedArgs &sa, const int32_t first_line, const int32_t item, Entry<PACKED> *stage_of_wave)
{
    constexpr int kAhead = VPL >= 3 ? 2 : 8 / VPL;          // steps in flight: 6 to 8 KB per wave
    constexpr int kRing = kAhead * kStep;                   // entries of a turn of the ring
    static_assert(kPart % kRing == 0 && kPart / kStep <= 64, "a part is a whole number of turns, a bit per step");
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
    // whole lines: from the slice's first line on, line v of a row in the instruction's offset; rows of any length: from the
    // first column on, and the lane's column in each line
    const int32_t begin = WHOLE ? first_line * kLine : 0;
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.H + begin), 0,
                                                        (int)buffer_extent(a.n_cols, a.ldh, begin), kRawBuffer);
    uint32_t lane_off[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v)
        lane_off[v] = WHOLE ? gl * 16 + v * kLine * 4 : (uint32_t)min(c0 + v * kLine, a.dim - 4) * 4;
    const auto packed_rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.p.packed), 0,
                                                               (int)(uint32_t)a.p.packed_bytes, kRawBuffer);
    const uint32_t pitch = (uint32_t)a.ldh * 4u;

    // After `sum_groups` lane l (and lane l + 32) holds column l of each line.
    const int line_col = lane & (kLine - 1);
    const int from_lane = ((line_col & 3) * 16 + line_col / 4) << 2;
    auto column_of = [&](int v) ADAQP_INLINE {                           // the column lane l holds a sum of; negative: none of its own
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
        uint64_t marks[2];                                  // bit s: a row ends in step s of the part, after one of its entries
    };
    int64_t r_hi;
    auto request_rows = [&](int32_t row) ADAQP_INLINE {
        const int64_t r = (int64_t)row + lane + 1;
        r_hi = a.rowptr[r < a.n_rows ? r : a.n_rows];
    };
    auto take = [&](int32_t row0, int64_t ent0) ADAQP_INLINE {           // from r_hi, requested for row0
        Chunk c;
        c.row0 = row0;
        c.ent0 = ent0;
        const int64_t end = clamp64(clamp64(r_hi, base, base + nnz_r) - base - ent0, 0, kNoEnd);
        c.ends = (int32_t)end;
        const int64_t left = j[1] - ent0;
        const int64_t most = kChunk - ((base + ent0) & (kLine - 1));       // up to a line of col and val
        c.n_ent = (int32_t)(left < most ? left : most);
        c.n_end = __popcll(__ballot(lane < kEnds && row0 + lane < i[1] && c.ends <= c.n_ent));
        if (c.n_end == kEnds) c.n_ent = min(c.n_ent, __builtin_amdgcn_readlane(c.ends, kEnds - 1));
        if (lane >= c.n_end) c.ends = kNoEnd;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int32_t last = c.ends - 1 - p * kPart;    // entry of the part that is its row's last
            const uint64_t mark = last >= 0 && last < kPart ? (uint64_t)1 << (last / kStep) : 0;
            c.marks[p] = (uint64_t)or_lanes((uint32_t)(mark >> 32)) << 32 | or_lanes((uint32_t)mark);
        }
        return c;
    };
    int4_t st_col[kLoads];
    float4_t st_val[kLoads];
    auto request_entries = [&](const Chunk &c) ADAQP_INLINE {            // past the chunk's entries: zeros
        const auto cols = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(a.col + base + c.ent0), 0, c.n_ent * 4, kRawBuffer);
        const auto vals = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.val + base + c.ent0), 0, c.n_ent * 4, kRawBuffer);
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {                  // streamed: keep the caches for H
            const int at = (k * kWave + lane) * 16;         // all of it here: the scalar offset is outside the range check
            st_col[k] = __builtin_bit_cast(int4_t, __builtin_amdgcn_raw_buffer_load_b128(cols, at, 0, kNonTemporal));
            st_val[k] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(vals, at, 0, kNonTemporal));
        }
    };
    auto stage = [&](const Chunk &c) ADAQP_INLINE {
        stage_entries<kLoads, PACKED>(st_col, st_val, c.n_ent, (uint32_t)a.n_cols, pitch, a.p, lane, stage_of_wave);
    };

    // the ring: kAhead steps whose lines are on their way
    float4_t h[kAhead][VPL];
    uint32_t words[kAhead][VPL], words_up[kAhead][VPL];     // four codes, where rows end anywhere across two words
    Entry<PACKED> in_flight[kAhead];
    auto packed_col = [&](int v) ADAQP_INLINE { return (uint32_t)a.p.col0 + (WHOLE ? (uint32_t)(c0 + v * kLine) : lane_off[v] / 4); };
    auto fetch = [&](auto tag, const Entry<PACKED> &en) ADAQP_INLINE {
        constexpr int U = decltype(tag)::value;
        in_flight[U] = en;
        const uint32_t w = PACKED ? en.off & 3u : 0u;
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const uint32_t off = PACKED && w != 0 ? kOutside : en.off + lane_off[v];
            h[U][v] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)off, 0, 0));
            if constexpr (PACKED) {
                words[U][v] = fetch_codes(packed_rows, en.off, packed_col(v), a.p.full_dim);
                if constexpr (!WHOLE) words_up[U][v] = fetch_codes(packed_rows, en.off, packed_col(v), a.p.full_dim, 1);
            }
        }
    };
    auto neighbour = [&](auto tag, int v) ADAQP_INLINE {                 // the four columns a lane fetched
        constexpr int U = decltype(tag)::value;
        float4_t x = h[U][v];
        if constexpr (PACKED) x = unpack_codes(in_flight[U], words[U][v], packed_col(v), x, WHOLE ? 0 : words_up[U][v]);
        return x;
    };

    // Sums of the open row: acc what the present chunk has given so far, per group; before what earlier chunks of the share
    // gave, as `sum_groups` leaves it.  No addition chain is longer than the 48 steps of half a chunk, the halves of a share's
    // chunks, or the shares of a row (one running sum over a share would be thousands of terms long and rounds accordingly).
    float4_t acc[VPL];
    float before[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        before[v] = 0.0f;
    }
    auto take_sums = [&](float (&sum)[VPL]) {               // and start anew
        sum_groups(acc, sum);
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            sum[v] = before[v] + sum[v];
            before[v] = 0.0f;
            acc[v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    auto keep_sums = [&]() ADAQP_INLINE {
        float sum[VPL];
        take_sums(sum);
#pragma unroll
        for (int v = 0; v < VPL; ++v) before[v] = sum[v];
    };
    float *out_row = a.out + (int64_t)i[0] * a.ldo;         // the rows of a share end one after the other
    // Lanes without a column of their own store outside the row's buffer: a branch around the store would be one the compiler
    // cannot take for uniform, and cost every step of the ring copies of the sums and a second jump.
    uint32_t store_at[VPL];
#pragma unroll
    for (int v = 0; v < VPL; ++v)
        store_at[v] = lane < kLine && column_of(v) >= 0 ? (uint32_t)column_of(v) * 4u : kOutside;
    auto store_row = [&](float *row, const float (&sum)[VPL], auto policy) {
        const auto to = __builtin_amdgcn_make_buffer_rsrc(row, 0, a.wdim * 4, kRawBuffer);
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sum[v]), to, (int)store_at[v], 0, decltype(policy)::value);
    };
    auto finish_row = [&]() ADAQP_INLINE {
        float sum[VPL];
        take_sums(sum);
        if constexpr (WHOLE) {
#pragma unroll
            for (int v = 0; v < VPL; ++v) sum[v] = column_of(v) < a.dim ? sum[v] : 0.0f;
            store_row(out_row, sum, std::integral_constant<int, kNonTemporal>());
        } else {                                            // lines are shared with other rows: left for the L2 to merge
            store_row(out_row, sum, std::integral_constant<int, 0>());
        }
        out_row += a.ldo;
    };

    // The walk starts behind a chunk of nothing, whose one turn finds an empty ring and fills it: staging and the first fetches
    // would be a second copy of that code, which a short launch pays for in instruction fetches.
    request_rows(i[0]);
    Chunk cur = {i[0], 0, 0, j[0], kNoEnd, {0, 0}};
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        in_flight[u] = {};
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            h[u][v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            words[u][v] = words_up[u][v] = 0;
        }
    }
    for (;;) {
        const int32_t next_row = cur.row0 + cur.n_end;
        const int64_t next_ent = cur.ent0 + cur.n_ent;
        Chunk next = take(next_row, next_ent);
        const bool more = next.n_end > 0 || next.n_ent > 0;
        if (more) {
            request_entries(next);
            request_rows(next.row0 + next.n_end);
        }
        int32_t e = 0;                                      // row ends behind us
        while (__builtin_amdgcn_readlane(cur.ends, e) == 0) {   // that belong to what the chunks before have added up
            finish_row();
            ++e;
        }
        const int32_t turns = cur.n_ent > 0 ? (cur.n_ent + kRing - 1) / kRing : 1;
        uint64_t marks = cur.marks[0];
        for (int32_t t = 0; t < turns; ++t) {
            if (t == kPart / kRing) {                       // the chunk's second part
                keep_sums();
                marks = cur.marks[1];
            }
            const Entry<PACKED> *src = stage_of_wave + (t + 1) * kRing + grp;
            if (t + 1 == turns) {                           // the ring goes on in the next chunk: all of this one has been read
                if (more) stage(next);
                else if (lane < kRing) stage_of_wave[lane] = Entry<PACKED>{kOutside, 0.0f};
                src = stage_of_wave + grp;
            }
            Entry<PACKED> en[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) en[u] = src[u * kStep];
            __builtin_amdgcn_sched_barrier(0);
            unroll<0, kAhead>([&](auto tag) {
                constexpr int U = decltype(tag)::value;
                float4_t x[VPL];
                float val = in_flight[U].val;
#pragma unroll
                for (int v = 0; v < VPL; ++v) x[v] = neighbour(tag, v);
                if ((uint32_t)marks & (1u << U)) {
                    // the groups from the last end to this one belong to the row that ends here
                    const int32_t at = (t * kAhead + U) * kStep;
                    int32_t from = 0, to = __builtin_amdgcn_readlane(cur.ends, e) - at;
                    do {
                        const bool mine = grp >= from && grp < to;
#pragma unroll
                        for (int v = 0; v < VPL; ++v)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const float sum = fmaf(val, x[v][k], acc[v][k]);
                                acc[v][k] = mine ? sum : acc[v][k];
                            }
                        finish_row();
                        ++e;
                        from = to;
                        to = __builtin_amdgcn_readlane(cur.ends, e) - at;
                    } while (to <= kStep);
                    // what is left is the next row's; no else: the sums would be copied where two branches meet
                    val = grp >= from ? val : 0.0f;
#pragma unroll
                    for (int v = 0; v < VPL; ++v)
#pragma unroll
                        for (int k = 0; k < 4; ++k) x[v][k] = grp >= from ? x[v][k] : 0.0f;
                }
#pragma unroll
                for (int v = 0; v < VPL; ++v)
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc[v][k] = fmaf(val, x[v][k], acc[v][k]);
                fetch(tag, en[U]);
                __builtin_amdgcn_sched_barrier(0);
            });
            marks >>= kAhead;
        }
        if (!more) break;
        keep_sums();                                        // the open row goes on in the next chunk
        cur = next;
    }
    // what is left belongs to a row that goes on in the next wave's share
    const int64_t began = i[1] < a.n_rows ? clamp64(a.rowptr[i[1]], base, base + nnz_r) - base : nnz_r;
    const bool held = i[1] < a.n_rows && j[1] > (began > j[0] ? began : j[0]);
    if (held) {
        float sum[VPL];
        take_sums(sum);
        store_row(a.carry + (int64_t)item * a.carry_ld, sum, std::integral_constant<int, 0>());
    }
    if (first_line == 0 && lane == 0) a.carry_row[item] = held ? i[1] : -1;
}

template <int VPL, bool PACKED, bool WHOLE>
__global__ __launch_bounds__(kBlock, 2) void spmm_sliced_kernel(const SlicedArgs sa)
{
    __shared__ alignas(16) Entry<PACKED> stages[kWavesPerBlock][kChunk];
    const SliceTasks tasks(sa.lines, VPL, sa.n_blocks, PACKED);
    const int32_t xcd = blockIdx.x % kXcds;
    const int64_t task = tasks.first_task(xcd) + blockIdx.x / kXcds;
    if (task >= tasks.first_task(xcd + 1)) return;
    const int32_t slice = (int32_t)(task / sa.n_blocks), blk = (int32_t)(task % sa.n_blocks);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t item = blk * kWavesPerBlock + wave;
    const int live = min(VPL, sa.lines - slice * VPL);
    if (live == VPL) walk_share<VPL, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 3) if (live == 3) walk_share<3, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 2) if (live == 2) walk_share<2, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 1) if (live == 1) walk_share<1, PACKED, WHOLE>(sa, slice * VPL, item, stages[wave]);
}

}  // namespace

SlicedCut plan_sliced(const SpmmArgs &a, int64_t nnz_hint, bool whole_lines, bool skewed_columns)
{
    if (!sliced_takes(a.n_rows, a.nnz, a.n_cols, a.ldh, a.p.slot_of_row != nullptr, a.p.packed_bytes, a.p.full_dim)) return {0, 0, 0};
    if (!whole_lines && a.dim < 4) return {0, 0, 0};        // a lane takes four columns
    return sliced_cut(a.n_rows, nnz_hint, a.n_cols, (a.wdim + kLine - 1) / kLine, whole_lines, skewed_columns);
}

hipError_t launch_sliced(const SpmmArgs &a, const SlicedCut &cut, int64_t nnz_hint, bool whole_lines, hipStream_t st,
                         int32_t *n_carries_out)
{
    SlicedArgs sa;
    sa.s = a;
    sa.lines = (a.wdim + kLine - 1) / kLine;
    const int vpl = a.p.slot_of_row ? cut.packed_lines : cut.lines;
    // each wave takes one share, of at least 256 steps of the path: a search and an empty ring each
    const int64_t path = nnz_hint + (int64_t)a.n_rows * kRowSteps;
    int64_t n_blocks = std::min(cut.n_blocks, (path + kMinPath - 1) / kMinPath);
    if (n_blocks > a.n_items / kWavesPerBlock) n_blocks = a.n_items / kWavesPerBlock;      // one carry slot per share
    if (n_blocks < 1) n_blocks = 1;
    sa.n_blocks = (int32_t)n_blocks;
    const dim3 grid((unsigned)(SliceTasks(sa.lines, vpl, sa.n_blocks, a.p.slot_of_row != nullptr).most_per_xcd() * kXcds));
#define ADAQP_SLICED(V, WHOLE)                                                                                   \
    do {                                                                                                         \
        if (a.p.slot_of_row) hipLaunchKernelGGL((spmm_sliced_kernel<V, true, WHOLE>), grid, dim3(kBlock), 0, st, sa); \
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
