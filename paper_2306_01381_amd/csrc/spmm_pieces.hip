// Neighbour aggregation (Sec. 2.1 Eq. 3) over a planned walk: the segments of rows in the order of column tiles, cut into pieces by the
// host.  A wave takes one piece for one slice of VPL lines of H and gathers as spmm_sliced.hip does: one load per line for eight
// entries, AHEAD steps of eight in flight, sums folded over the eight groups where a segment ends.
//
// What bounds the gathers of segments is what their group of tiles misses in the L2, and that hangs on how far apart the entries are
// that an XCD has under way.  Shares cut on the device are a search each (eight loads that wait for one another, 20 us under load)
// and so have to be long: 128 workgroups with 4 600 entries each span two groups, 13 % of the lines come from behind the L2, and the
// L1, which answers in order, stands still for each of them (31 % of its time).  A planned piece begins with one load of its bounds and
// is 700 entries long; workgroups start in order, so that those under way are neighbours: 5.7 % from behind the L2, 24 %.
// Waves that take piece after piece drift apart and lose that (28 % from behind the L2, 1.29 -> 1.55 ms for the step below).
// A piece is one LDS fill, so nothing of the next has to wait in registers: 75 of them, and no spilled scalars.
//
// 58 000 rows, 27.8 M entries, 98 000 columns, 256 columns of H, the whole layer step: shares 1.40 ms, here with as many waves as
// registers allow 1.29, with 16 per CU 1.19 (25 TB/s of gathers; bare loads out of the L2 31; 24 waves of two lines ask for more
// than their group; two lines per slice 1.19, one 1.46, four 1.31).  306 000 rows, 7.7 M entries, 456 000 columns, whose groups
// are three times an L2: shares 1.04 ms, two lines per slice 0.83, one 0.75.
#include <algorithm>
#include <new>
#include <vector>

#include "spmm_common.hpp"
#include "spmm_wave.hpp"

namespace adaqp {
namespace {

constexpr int kEntries = ADAQP_SPMM_PIECE_ENTRIES;
constexpr int kEnds = ADAQP_SPMM_PIECE_SEGMENTS;
constexpr int kPart = 256, kParts = kEntries / kPart;       // no sum runs longer than a part's 32 steps
constexpr int kLoads = kEntries / (4 * kWave);              // of four entries per lane: what a piece takes of col, and of val
constexpr int32_t kNoEnd = 0x10000;                         // lies after every step of a piece
constexpr unsigned kIdleLds = 6144;                         // of a workgroup, beside its 26 KB: no more than 16 waves on a CU
constexpr int64_t kMostPieces = 1 << 24, kMostTasks = 1 << 23;
static_assert(kEnds < kWave - 1, "a lane per end, and one that has none");

struct alignas(8) Entry { uint32_t off; float val; };       // byte offset of a row of H, coefficient

template <int VPL, int AHEAD>
__device__ __forceinline__ void walk_piece(const PieceArgs &a, const int32_t first_line, const int32_t item, Entry *stage)
{
    constexpr int kRing = AHEAD * kStep;                    // entries of a turn of the ring
    static_assert(kPart % kRing == 0 && kEntries % kPart == 0 && kPart / kStep <= 32, "a part is a whole number of turns, a bit per step");
    const int lane = threadIdx.x & (kWave - 1), gl = lane & (kGroup - 1), grp = lane / kGroup;

    const adaqp_spmm_piece from = a.pieces[item], to = a.pieces[item + 1];
    const int32_t seg0 = min(max(from.segment, 0), a.n_seg);
    const int32_t n_end = min(max(to.segment - seg0, 0), min(a.n_seg - seg0, kEnds));
    const int64_t ent0 = clamp64(from.entry, 0, a.n_entries);
    const int32_t n_ent = (int32_t)clamp64(to.entry - ent0, 0, min((int64_t)kEntries, a.n_entries - ent0));
    // steps are counted so that the last turn of the ring is a full one: a fetch of nothing takes as long as one of a line
    const int32_t n_steps = (n_ent + kStep - 1) / kStep, turns = (n_steps + AHEAD - 1) / AHEAD, pad = turns * AHEAD - n_steps;

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
    int32_t ends = kNoEnd, dests = 0;                       // lane l: where segment seg0 + l ends, and where its sum goes
    if (lane < n_end) {
        ends = (int32_t)clamp64(a.ptr[(int64_t)seg0 + lane + 1] - ent0, 0, n_ent) + pad * kStep;
        dests = a.dest[seg0 + lane];
    }

    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.H + first_line * kLine), 0,
                                                        (int)buffer_extent(a.n_cols, a.ldh, first_line * kLine), kRawBuffer);
    const uint32_t pitch = (uint32_t)a.ldh * 4u;
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            float4_t two;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bool ok = (k * kWave + lane) * 4 + q + r < n_ent && (uint32_t)st_col[k][q + r] < (uint32_t)a.n_cols;
                two[2 * r] = __builtin_bit_cast(float, ok ? (uint32_t)st_col[k][q + r] * pitch : kOutside);     // else: fetches nothing
                two[2 * r + 1] = ok ? st_val[k][q + r] : 0.0f;
            }
            *reinterpret_cast<float4_t *>(stage + pad * kStep + (k * kWave + lane) * 4 + q) = two;
        }
    uint32_t marks[kParts];                                 // bit s: a segment ends in step s of the part, after one of its entries
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
        const int32_t last = ends - 1 - p * kPart;
        marks[p] = or_lanes(last >= 0 && last < kPart ? 1u << (last / kStep) : 0u);
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
    // Lanes without a column of their own store outside the row's buffer: no branch.
    const uint32_t store_at = lane < kLine ? (uint32_t)(first_line * kLine + lane) * 4u : kOutside;
    auto store_sums = [&](int32_t dest) ADAQP_INLINE {      // partial row, or -1 - row
        float sum[VPL];
        take_sums(sum);
        const bool part = dest >= 0, known = part ? dest < a.n_partials : -1 - dest < a.n_rows;
        float *row = part ? a.partial + (int64_t)dest * a.ldp : a.out + (int64_t)(-1 - dest) * a.ldo;
        const auto to_row = __builtin_amdgcn_make_buffer_rsrc(row, 0, known ? a.wdim * 4 : 0, kRawBuffer);
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
            const float x = (first_line + v) * kLine + line_col < a.dim ? sum[v] : 0.0f;        // row padding
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), to_row, (int)store_at + v * kLine * 4, 0, kNonTemporal);
        }
    };

    // the ring: AHEAD steps whose lines are on their way
    float4_t h[AHEAD][VPL];
    float w[AHEAD];
    const uint32_t lane_off = gl * 16;
    auto fetch = [&](auto tag, const Entry &en) ADAQP_INLINE {
        constexpr int U = decltype(tag)::value;
        w[U] = en.val;
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            h[U][v] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(en.off + lane_off + v * kLine * 4), 0, 0));
    };
    unroll<0, AHEAD>([&](auto tag) ADAQP_INLINE {
        constexpr int U = decltype(tag)::value;
        if (U >= pad) {
            fetch(tag, stage[U * kStep + grp]);
        } else {
            w[U] = 0.0f;
#pragma unroll
            for (int v = 0; v < VPL; ++v) h[U][v] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
    });
    int32_t e = 0;                                          // segment ends behind us
    while (__builtin_amdgcn_readlane(ends, e) <= pad * kStep) {      // segments without entries
        store_sums(__builtin_amdgcn_readlane(dests, e));
        ++e;
    }
    auto turn = [&](int32_t t, auto goes_on) ADAQP_INLINE {
        constexpr bool kGoesOn = decltype(goes_on)::value;  // else: the last one, whose lines are the last
        if (t > 0 && t % (kPart / kRing) == 0) {            // the next part
#pragma unroll
            for (int p = 0; p + 1 < kParts; ++p) marks[p] = marks[p + 1];
            float sum[VPL];
            take_sums(sum);
#pragma unroll
            for (int v = 0; v < VPL; ++v) before[v] = sum[v];
        }
        Entry en[AHEAD];
        if constexpr (kGoesOn)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) en[u] = stage[(t + 1) * kRing + u * kStep + grp];
        __builtin_amdgcn_sched_barrier(0);
        unroll<0, AHEAD>([&](auto tag) ADAQP_INLINE {
            constexpr int U = decltype(tag)::value;
            float4_t x[VPL];
            float val = w[U];
#pragma unroll
            for (int v = 0; v < VPL; ++v) x[v] = h[U][v];
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
                    store_sums(__builtin_amdgcn_readlane(dests, e));
                    ++e;
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
    int32_t t = 0;
    for (; t + 1 < turns; ++t) turn(t, std::true_type());
    if (t < turns) turn(t, std::false_type());
    if (to.partial >= 0) store_sums(to.partial);            // of a segment that goes on in the next piece
}

template <int VPL, int AHEAD>
__global__ __launch_bounds__(kBlock, 4) void spmm_pieces_kernel(const PieceArgs a)
{
    __shared__ alignas(16) Entry stages[kWavesPerBlock][kEntries + kWave];
    const SliceTasks tasks(a.lines, VPL, a.n_blocks, false);
    const int32_t xcd = blockIdx.x % kXcds;
    const int64_t task = tasks.first_task(xcd) + blockIdx.x / kXcds;
    if (task >= tasks.first_task(xcd + 1)) return;
    const int32_t slice = (int32_t)(task / a.n_blocks), blk = (int32_t)(task % a.n_blocks);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t item = blk * kWavesPerBlock + wave;
    if (item >= a.n_pieces) return;
    const int live = min(VPL, a.lines - slice * VPL);
    if (live == VPL) walk_piece<VPL, AHEAD>(a, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 3) if (live == 3) walk_piece<3, AHEAD>(a, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 2) if (live == 2) walk_piece<2, 2 * AHEAD>(a, slice * VPL, item, stages[wave]);
    if constexpr (VPL > 1) if (live == 1) walk_piece<1, 8>(a, slice * VPL, item, stages[wave]);
}

// out[row] = sum of the row's partial rows in order; whole lines, row padding zero.  A wave per row, eight partial rows of a strip of 256
// columns in flight together (28 000 rows of eight, 256 columns: 42 us, 6.1 TB/s).  Rows of one segment need none: of 306 000 rows
// one in twelve has two (129 -> 20 us).
__global__ __launch_bounds__(kBlock) void pieces_sum_kernel(const int32_t *sum_row, const int32_t *sum_ptr, int64_t n_sums, int32_t n_partials,
                                                            const float *partial, int32_t dim, int64_t wdim, float *out, int64_t ldo, int32_t n_rows)
{
    constexpr int kAhead = 8;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t s = (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (s >= n_sums) return;
    const int32_t row = sum_row[s], from = max(0, sum_ptr[s]), end = min(sum_ptr[s + 1], n_partials);
    if (row < 0 || row >= n_rows) return;
    for (int64_t c = lane * 4; c < wdim; c += kWave * 4) {
        float4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int32_t p = from; p < end; p += kAhead) {
            float4_t x[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                x[q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                if (p + q < end) x[q] = __builtin_nontemporal_load(reinterpret_cast<const float4_t *>(partial + (int64_t)(p + q) * wdim + c));
            }
#pragma unroll
            for (int q = 0; q < kAhead; ++q) sum += x[q];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k >= dim) sum[k] = 0.0f;
        __builtin_nontemporal_store(sum, reinterpret_cast<float4_t *>(out + (int64_t)row * ldo + c));
    }
}

// Length of a piece in entries and eight times ends of segments: eight pieces and more for each of the 4 096 waves that are under way
// (2.5 M entries, 602 columns), and no longer than pays.  A start costs 0.2 us of its CU (28 M entries, 256 columns, two lines: 320 long
// 1.37 ms, 512 1.19, 864 1.19; 7.7 M entries, one line: 320 0.765, 448 0.753, 524 0.767).
int64_t piece_length(int64_t n_seg, int64_t n_entries, int32_t dim, int32_t lines_per_slice)
{
    const int64_t slices = ((int64_t)dim + 32 * lines_per_slice - 1) / (32 * lines_per_slice), path = n_entries + 8 * n_seg;
    return std::min<int64_t>(std::max<int64_t>(path / 32768 * slices, 128), lines_per_slice == 1 ? 448 : kEntries + 96);
}

}  // namespace

int check_pieces(const adaqp_spmm_pieces *p, int64_t n_seg)
{
    if (p->n_pieces < 0 || p->n_partials < 0 || p->n_sums < 0 || n_seg < 0) return ADAQP_EINVAL;
    if (p->n_pieces == 0) return ADAQP_OK;
    if (p->n_pieces > kMostPieces || p->n_partials > INT32_MAX - 1024 || p->n_sums > INT32_MAX - 1024) return ADAQP_ESIZE;
    if (p->lines_per_slice != 1 && p->lines_per_slice != 2 && p->lines_per_slice != 4) return ADAQP_EINVAL;
    if (!p->pieces_dev || !p->sum_ptr_dev || (n_seg > 0 && !p->dest_dev) || (p->n_sums > 0 && !p->sum_row_dev)) return ADAQP_EINVAL;
    if (!aligned_to(p->pieces_dev, 16) || !aligned_to(p->dest_dev, 4) || !aligned_to(p->sum_row_dev, 4) || !aligned_to(p->sum_ptr_dev, 4)) return ADAQP_EINVAL;
    return ADAQP_OK;
}

int launch_pieces(const adaqp_spmm_pieces *p, PieceArgs a, hipStream_t st)
{
    a.pieces = p->pieces_dev;
    a.dest = p->dest_dev;
    a.n_pieces = (int32_t)p->n_pieces;
    a.n_partials = (int32_t)p->n_partials;
    a.ldp = ((int64_t)a.dim + kLine - 1) / kLine * kLine;
    a.n_blocks = (a.n_pieces + kWavesPerBlock - 1) / kWavesPerBlock;
    // a launch has fewer than 2^32 threads: as many slices as that allows
    const int64_t most_lines = std::max<int64_t>(kMostTasks / a.n_blocks, 1) * p->lines_per_slice, lines = a.ldp / kLine;
    for (int64_t l0 = 0; l0 < lines; l0 += most_lines) {
        PieceArgs s = a;
        s.lines = (int32_t)std::min(lines - l0, most_lines);
        s.dim = (int32_t)std::min<int64_t>(a.dim - l0 * kLine, (int64_t)s.lines * kLine);
        s.wdim = s.lines * kLine;
        s.H += l0 * kLine;
        s.out += l0 * kLine;
        if (s.partial) s.partial += l0 * kLine;
        const dim3 grid((unsigned)(SliceTasks(s.lines, p->lines_per_slice, s.n_blocks, false).most_per_xcd() * kXcds));
        if (p->lines_per_slice == 1) hipLaunchKernelGGL((spmm_pieces_kernel<1, 8>), grid, dim3(kBlock), 0, st, s);
        else if (p->lines_per_slice == 2) hipLaunchKernelGGL((spmm_pieces_kernel<2, 4>), grid, dim3(kBlock), kIdleLds, st, s);
        else hipLaunchKernelGGL((spmm_pieces_kernel<4, 2>), grid, dim3(kBlock), kIdleLds, st, s);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    constexpr int64_t kMostSums = (int64_t)1 << 24;         // of a launch, for the same reason
    for (int64_t s0 = 0; s0 < p->n_sums; s0 += kMostSums) {
        const int64_t n = std::min(p->n_sums - s0, kMostSums);
        hipLaunchKernelGGL(pieces_sum_kernel, dim3((unsigned)((n + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(kBlock), 0, st, p->sum_row_dev + s0,
                           p->sum_ptr_dev + s0, n, a.n_partials, a.partial, a.dim, a.ldp, a.out, a.ldo, a.n_rows);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    return ADAQP_OK;
}

}  // namespace adaqp

using namespace adaqp;

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
    if (n_seg < 0 || n_rows < 0 || dim <= 0 || !ptr_host || !sizes_inout || ptr_host[0] < 0 || (n_rows > 0 && !of_row_host)) return ADAQP_EINVAL;
    if (lines_per_slice != 1 && lines_per_slice != 2 && lines_per_slice != 4) return ADAQP_EINVAL;
    if (n_seg > INT32_MAX - 1024 || n_rows > INT32_MAX - 1024) return ADAQP_ESIZE;
    const bool fill = pieces_out != nullptr;
    if (fill && ((n_seg > 0 && !dest_out) || !sum_ptr_out || (sizes_inout[2] > 0 && !sum_row_out))) return ADAQP_EINVAL;
    for (int64_t s = 0; s < n_seg; ++s)
        if (ptr_host[s + 1] < ptr_host[s]) return ADAQP_EINVAL;
    const int64_t last = ptr_host[n_seg], length = piece_length(n_seg, last - ptr_host[0], dim, lines_per_slice);

    // Pieces of whole segments; one that would be less than half full takes the next segment up to a line of entries.
    std::vector<adaqp_spmm_piece> pieces{{ptr_host[0], 0, -1}};
    std::vector<int32_t> cuts((size_t)n_seg, 0);            // of a segment
    for (int64_t seg = 0, entry = ptr_host[0]; seg < n_seg;) {
        const int64_t first_seg = seg, first = entry;
        auto weight = [&](int64_t e, int64_t s) { return e - first + 8 * (s - first_seg); };
        while (seg < n_seg && seg - first_seg < kEnds && ptr_host[seg + 1] - first <= kEntries && weight(ptr_host[seg + 1], seg + 1) <= length)
            entry = ptr_host[++seg];
        int32_t partial = -1;
        if (seg < n_seg && seg - first_seg < kEnds && weight(entry, seg) < length / 2) {
            const int64_t to = (first + std::min<int64_t>(length - 8 * (seg - first_seg), kEntries)) / 32 * 32;
            if (to > entry && to < ptr_host[seg + 1]) {
                entry = to;
                partial = cuts[(size_t)seg]++;
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
        const int32_t *of = of_row_host + r * S;
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
    const int64_t sizes[3] = {(int64_t)pieces.size() - 1, n_partials, (int64_t)sum_row.size()};
    if (!fill) {
        std::copy(sizes, sizes + 3, sizes_inout);
        return ADAQP_OK;
    }
    if (!std::equal(sizes, sizes + 3, sizes_inout)) return ADAQP_EINVAL;
    std::copy(pieces.begin(), pieces.end(), pieces_out);
    std::copy(dest.begin(), dest.end(), dest_out);
    std::copy(sum_row.begin(), sum_row.end(), sum_row_out);
    std::copy(sum_ptr.begin(), sum_ptr.end(), sum_ptr_out);
    return ADAQP_OK;
} catch (const std::bad_alloc &) {           // nothing may be thrown through a C entry
    return ADAQP_ESIZE;
}
