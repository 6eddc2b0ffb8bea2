// Neighbour aggregation out_v = sum_u alpha(u,v) h_u (Sec. 2.1 Eq. 3, inner sum) as a CSR SpMM for gfx950.
//
// Work split.  Degrees follow a power law (the largest row is ~50x the mean), so rows are not the unit of
// work.  The CSR is walked as a merge path: the list of row ends and the list of entries are merged, the
// path of length n_rows + nnz is cut into equal pieces, one piece per wave.  A wave finds its two end points
// with a 64-ary search over rowptr (every lane probes one position), then walks its piece:
//   * entries are staged 64 at a time, lane e holding (col, alpha) of entry e; the wave-uniform column of
//     the entry being processed is fetched with v_readlane, so the neighbour row's address is scalar and
//     every lane loads its VW-float slice of that row with one vector load;
//   * row ends are staged the same way, 64 rows at a time;
//   * U entries are in flight at once (U * NV vector loads per lane) before the first is consumed;
//   * a row that ends inside the piece is stored directly; what a piece has accumulated for a row that
//     continues into the next piece goes to a carry slot in the workspace, or (merge_joins, spmm_rules.hpp) meets the rest of the row in LDS,
//     where that is a piece of the same workgroup, and a workgroup has a carry slot for the row that continues in the next one.
// A second, tiny kernel adds the carries of each split row in order.  The summation order therefore
// depends only on the launch geometry: results are bit-identical from run to run and across schedules.
//
// Where sliced_cut (spmm_rules.hpp) says so the kernel of spmm_sliced.hip takes the call instead (same path, feature columns
// sliced over the XCDs); this one serves launches of few entries, short rows that slices fit badly, most rows that share
// lines, and matrices too large for that kernel's 32-bit offsets.
//
// The kernel is a gather: per entry it reads 8 bytes of (col, alpha) and 4*dim bytes of H.  It is bound by
// how fast H rows come out of L2 / Infinity Cache / HBM, not by arithmetic, so there is no MFMA use.
#include <algorithm>
#include <cmath>
#include <functional>
#include <mutex>
#include <new>
#include <numeric>
#include <vector>

#include "spmm_common.hpp"

namespace adaqp {
namespace {

template <int VW> struct VecOf;
template <> struct VecOf<1> { using type = float; };
template <> struct VecOf<2> { using type = float2; };
template <> struct VecOf<4> { using type = float4; };

template <int VW>
__device__ __forceinline__ void load_vec(const float *p, float *dst)
{
    using V = typename VecOf<VW>::type;
    const V v = *reinterpret_cast<const V *>(p);
    if constexpr (VW == 1) { dst[0] = v; }
    if constexpr (VW == 2) { dst[0] = v.x; dst[1] = v.y; }
    if constexpr (VW == 4) { dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w; }
}

template <int VW>
__device__ __forceinline__ void store_vec(float *p, const float *src)
{
    using V = typename VecOf<VW>::type;
    if constexpr (VW == 1) { *p = src[0]; }
    if constexpr (VW == 2) { *reinterpret_cast<V *>(p) = make_float2(src[0], src[1]); }
    if constexpr (VW == 4) { *reinterpret_cast<V *>(p) = make_float4(src[0], src[1], src[2], src[3]); }
}

// Same, marked non-temporal: output rows are written once and not read again by this kernel.
template <int VW>
__device__ __forceinline__ void store_vec_streaming(float *p, const float *src)
{
    typedef float vec_t __attribute__((ext_vector_type(VW)));
    vec_t v;
    for (int k = 0; k < VW; ++k) v[k] = src[k];
    __builtin_nontemporal_store(v, reinterpret_cast<vec_t *>(p));
}

__device__ __forceinline__ int32_t uniform_i32(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ int64_t uniform_i64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int lane_id)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)v, lane_id);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)((uint64_t)v >> 32), lane_id);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Merge-path split point on diagonal d: the number of row ends that precede d path steps.  Row end i (its
// entry count relative to the range is end_i) precedes entry j iff end_i <= j; on diagonal d this reads
// end_i + i + 1 <= d, which is increasing in i, so the answer is the first i for which it fails.
// All 64 lanes take part; the result is wave-uniform.
__device__ int64_t split_rows(const SpmmArgs &a, int64_t d, int64_t base, int64_t nnz_r, int lane)
{
    int64_t lo = d - nnz_r > 0 ? d - nnz_r : 0;
    int64_t hi = d < a.n_rows ? d : a.n_rows;
    while (lo < hi) {
        const int64_t n = hi - lo;
        const int64_t step = (n + kWave - 1) / kWave;
        const int64_t probes = (n + step - 1) / step;          // <= 64
        const int64_t p = lo + lane * step;
        bool before = false;
        if (lane < probes) {
            const int64_t end_p = clamp64(a.rowptr[p + 1], base, base + nnz_r) - base;
            before = end_p + p + 1 <= d;
        }
        const int cnt = __popcll(__ballot(before));
        const int64_t new_lo = cnt > 0 ? lo + (int64_t)(cnt - 1) * step + 1 : lo;
        const int64_t new_hi = cnt < probes ? lo + (int64_t)cnt * step : hi;
        lo = new_lo;
        hi = new_hi;
    }
    return lo;
}

constexpr int32_t kNoRow = -1;
constexpr int32_t kFar = 0x7FFFFFFF;

// PACKED: entries whose column has a slot in slot_of_row take the neighbour row from the packed receive buffer
// and de-quantise it in registers, (float)code * S + Z as in Sec. 2.3 Eq. 5 (product rounded, then sum rounded),
// so the result is bit-identical to de-quantising into H first - without writing and re-reading those rows.
//
// JOINS: nearly every piece leaves a part of a row to the next one.  As long as a row's parts and ends lie in one workgroup they are added up
// in its LDS, and there is a carry slot per workgroup instead of one per piece (send, receive and sums of 60 000 rows, 1 M entries, 301
// columns 213 -> 201 us, of it the carries 17 -> 7; 150 000 rows, 1.2 M, 472 columns 440 -> 404; error against 64 bits 0.98 times, never more,
// over 14 graphs).  Parts are read whole and all open rows at once: column by column, with a wait for each, small calls took 1.04 times as long
// (462 calls 1.02).  Rows of more floats per lane leave a carry per piece.  Joining up to 16 would keep no workgroup away (registers allow
// fewer of them than 33 KB of LDS each) and was faster where it was timed, 602 columns 368 -> 346 us, 1 000 columns 387 -> 367.
constexpr int kJoinFloats = 8;              // of a lane, per row: 16 KB for a workgroup's parts and first rows

template <int VW, int NV, int U, bool PACKED, bool CHAINS, bool JOINS>
__global__ __launch_bounds__(kBlock) void spmm_merge_kernel(const SpmmArgs a)
{
    static_assert(!JOINS || VW * NV <= kJoinFloats);
    constexpr int kPartFloats = JOINS ? NV * kWave * VW : 1;
    __shared__ alignas(16) float open[JOINS ? kWavesPerBlock : 1][kPartFloats];         // what a piece has of the row that it leaves open
    __shared__ alignas(16) float first[JOINS ? kWavesPerBlock : 1][kPartFloats];        // and of the first row that ends in it
    __shared__ alignas(16) int32_t open_row[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1), wave = uniform_i32((int32_t)(threadIdx.x >> 6));
    const int32_t item = uniform_i32((int32_t)(blockIdx.x * kWavesPerBlock) + wave);
    if (!JOINS && item >= a.n_items) return;

    // extent of the range on the device: the host only sized the launch
    const int64_t base = uniform_i64(clamp64(a.rowptr[0], 0, a.nnz));
    const int64_t nnz_r = uniform_i64(clamp64(a.rowptr[a.n_rows], base, a.nnz)) - base;
    const int64_t total = (int64_t)a.n_rows + nnz_r;
    const int64_t per = (total + a.n_items - 1) / a.n_items;
    const int64_t d0 = (int64_t)item * per < total ? (int64_t)item * per : total;
    const int64_t d1 = item < a.n_items && d0 + per < total ? d0 + per : (item < a.n_items ? total : d0);
    if (!JOINS && d0 >= d1) {
        if (lane == 0) a.carry_row[item] = kNoRow;
        return;
    }
    const int64_t i0 = uniform_i64(split_rows(a, d0, base, nnz_r, lane));
    const int64_t i1 = uniform_i64(split_rows(a, d1, base, nnz_r, lane));
    const int64_t j0 = d0 - i0;                             // first entry of the piece, relative to base
    const int32_t n_edges = (int32_t)((d1 - i1) - j0);      // entries in the piece

    // per-lane slice of a row: vectors v*64 + lane, v < NV; only the last one can fall off the row
    const bool last_ok = ((NV - 1) * kWave + lane) * VW < a.wdim;

    // CHAINS: a row's sum is what it had at the piece's last multiple of kChain entries, and what came since, so that in long pieces no
    // chain of roundings is longer than in pieces of 32 steps (one sum over 128: up to 1.28 times their error against 64 bits).
    constexpr int kChain = 32;
    static_assert(kChain % U == 0 && kWave % kChain == 0, "chains end between groups of loads");
    float acc[NV][VW], before[NV][VW];                      // (before: CHAINS)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < VW; ++k) acc[v][k] = before[v][k] = 0.0f;

    // row-end staging: lane q holds the end (relative to j0) of row row_blk + q
    int64_t row = i0, row_blk = i0;
    int32_t my_end = kFar;
    auto stage_rows = [&]() {
        my_end = kFar;
        const int64_t q = row_blk + lane;
        if (q < a.n_rows) {
            const int64_t e = clamp64(a.rowptr[q + 1], base, base + nnz_r) - base - j0;
            my_end = e > kFar ? kFar : (e < 0 ? 0 : (int32_t)e);
        }
    };
    stage_rows();
    int32_t cur_end = __builtin_amdgcn_readlane(my_end, 0);
    bool dirty = false;

    auto whole_sum = [&]() {
        if constexpr (CHAINS) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < VW; ++k) {
                    acc[v][k] += before[v][k];
                    before[v][k] = 0.0f;
                }
        }
    };
    auto store_row = [&](int64_t r, float (&sum)[NV][VW]) {
        float *o = a.out + r * a.ldo;
        if (a.wdim > a.dim) {                                   // row padding: whatever was gathered there is dropped
#pragma unroll
            for (int k = 0; k < VW; ++k)
                if (((NV - 1) * kWave + lane) * VW + k >= a.dim) sum[NV - 1][k] = 0.0f;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (v < NV - 1 || last_ok) store_vec_streaming<VW>(o + (v * kWave + lane) * VW, sum[v]);
    };
    auto to_lds = [&](float *to) {
        if constexpr (JOINS)
#pragma unroll
            for (int v = 0; v < NV; ++v) store_vec<VW>(to + (v * kWave + lane) * VW, acc[v]);
    };
    auto flush_row = [&]() {
        whole_sum();
        // other waves may have parts of the first one
        if (JOINS && wave > 0 && row == i0) to_lds(first[wave]);
        else store_row(row, acc);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int k = 0; k < VW; ++k) acc[v][k] = 0.0f;
        dirty = false;
        ++row;
        if (row - row_blk == kWave) {
            row_blk = row;
            stage_rows();
        }
        cur_end = __builtin_amdgcn_readlane(my_end, (int)(row - row_blk));
    };

    const int32_t *colp = a.col + base + j0;
    const float *valp = a.val + base + j0;
    int32_t j = 0;                                          // entries consumed, relative to j0
    while (j < n_edges) {
        const int32_t nb = n_edges - j < kWave ? n_edges - j : kWave;
        int32_t my_col = 0;
        float my_val = 0.0f;
        int32_t my_b = 0;                                   // PACKED: width of the entry's packed row, 0 = plain row
        int64_t my_off = 0;
        float my_z = 0.0f, my_s = 0.0f;
        if (lane < nb) {
            my_col = __builtin_nontemporal_load(colp + j + lane);     // streamed once: keep the caches for H
            my_val = __builtin_nontemporal_load(valp + j + lane);
            if (my_col < 0 || my_col >= a.n_cols) { my_col = 0; my_val = 0.0f; }   // out-of-range entry: skipped
            if (PACKED) {
                const int32_t slot = a.p.slot_of_row[my_col];
                if (slot >= 0 && slot < a.p.n_slots) {
                    my_b = a.p.bits[slot];
                    my_off = a.p.row_offset[slot];
                    const float2 zs = *reinterpret_cast<const float2 *>(a.p.params + 2 * (int64_t)slot);
                    my_z = zs.x;
                    my_s = zs.y;
                    const int64_t stride = 4 * (((int64_t)a.p.full_dim * my_b + 31) >> 5);
                    const bool ok = (my_b == 2 || my_b == 4 || my_b == 8) && my_off >= 0 && (my_off & 3) == 0 &&
                                    my_off + stride <= a.p.packed_bytes;
                    if (!ok) my_b = 0;                      // broken slot: fall back to the row in H
                }
            }
        }
        for (int32_t e = 0; e < nb; e += U) {
            if constexpr (CHAINS) {
                if (e % kChain == 0) {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int k = 0; k < VW; ++k) {
                            before[v][k] += acc[v][k];
                            acc[v][k] = 0.0f;
                        }
                }
            }
            float h[U][NV][VW];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t eu = e + u < nb ? e + u : nb - 1;                    // tail repeats the last entry
                const int32_t c = __builtin_amdgcn_readlane(my_col, eu);
                const int32_t pb = PACKED ? __builtin_amdgcn_readlane(my_b, eu) : 0;
                if (PACKED && pb != 0) {                                           // wave-uniform
                    // one 32-bit word holds the VW codes of a lane's vector (VW * b <= 32 and divides 32)
                    const uint32_t *words = reinterpret_cast<const uint32_t *>(a.p.packed + readlane_i64(my_off, eu));
                    const uint32_t last_word = (uint32_t)(((int64_t)a.p.full_dim * pb - 1) >> 5);
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const uint32_t bit = (uint32_t)(a.p.col0 + (v * kWave + lane) * VW) * (uint32_t)pb;
                        const uint32_t idx = (bit >> 5) < last_word ? (bit >> 5) : last_word;
#pragma unroll
                        for (int k = 0; k < VW; ++k) h[u][v][k] = 0.0f;
                        h[u][v][0] = __builtin_bit_cast(float, words[idx]);
                    }
                } else {
                    const float *hrow = a.H + (int64_t)c * a.ldh;
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        if (v < NV - 1 || last_ok) {
                            load_vec<VW>(hrow + (v * kWave + lane) * VW, h[u][v]);
                        } else {
#pragma unroll
                            for (int k = 0; k < VW; ++k) h[u][v][k] = 0.0f;
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e + u < nb) {
                    while (j >= cur_end && row < i1) flush_row();    // rows that end before this entry
                    const float alpha = __builtin_bit_cast(
                        float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, my_val), e + u));
                    const int32_t pb = PACKED ? __builtin_amdgcn_readlane(my_b, e + u) : 0;
                    if (PACKED && pb != 0) {
                        const float Z = __builtin_bit_cast(
                            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, my_z), e + u));
                        const float S = __builtin_bit_cast(
                            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, my_s), e + u));
                        const uint32_t mask = (1u << pb) - 1u;
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const uint32_t bit = (uint32_t)(a.p.col0 + (v * kWave + lane) * VW) * (uint32_t)pb;
                            const uint32_t word = __builtin_bit_cast(uint32_t, h[u][v][0]) >> (bit & 31u);
#pragma unroll
                            for (int k = 0; k < VW; ++k) {
                                const uint32_t code = (word >> (k * pb)) & mask;
                                const float scaled = (float)code * S;      // Eq. 5: product rounded, then sum rounded
                                const float value = scaled + Z;
                                acc[v][k] = fmaf(alpha, value, acc[v][k]);
                            }
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < NV; ++v)
#pragma unroll
                            for (int k = 0; k < VW; ++k) acc[v][k] = fmaf(alpha, h[u][v][k], acc[v][k]);
                    }
                    ++j;
                    dirty = true;
                }
            }
        }
    }
    while (row < i1) flush_row();                           // rows that end at the piece's last entry, empty rows

    // what is left belongs to a row that continues in the next piece
    const int32_t left = dirty && row < a.n_rows ? (int32_t)row : kNoRow;
    if (left != kNoRow) whole_sum();
    auto store_carry = [&](int32_t slot) {
        float *cslot = a.carry + (int64_t)slot * a.carry_ld;
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (v < NV - 1 || last_ok) store_vec<VW>(cslot + (v * kWave + lane) * VW, acc[v]);
    };
    if constexpr (!JOINS) {
        if (left != kNoRow) store_carry(item);
        if (lane == 0) a.carry_row[item] = left;
    } else {
        if (left != kNoRow) to_lds(open[wave]);
        if (lane == 0) open_row[wave] = left;
        __syncthreads();
        const int4 rows = *reinterpret_cast<const int4 *>(open_row);
        const int32_t left_open[kWavesPerBlock] = {uniform_i32(rows.x), uniform_i32(rows.y), uniform_i32(rows.z), uniform_i32(rows.w)};
        static_assert(kWavesPerBlock == 4, "open_row is read at once");
        auto add = [&](const float *part) {
            float x[NV][VW];
#pragma unroll
            for (int v = 0; v < NV; ++v) load_vec<VW>(part + (v * kWave + lane) * VW, x[v]);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < VW; ++k) acc[v][k] += x[v][k];
        };
        // acc = the parts of row r that the waves before `end` leave open, in order
        auto add_open = [&](int32_t r, int end) {
            int begin = end;
#pragma unroll
            for (int w = kWavesPerBlock - 1; w >= 0; --w)
                if (begin == w + 1 && left_open[w] == r) begin = w;
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < VW; ++k) acc[v][k] = 0.0f;
            for (int w = begin; w < end; ++w) add(open[w]);
        };
        if (wave > 0 && i1 > i0) {
            add_open((int32_t)i0, wave);
            add(first[wave]);
            store_row(i0, acc);
        }
        if (wave == kWavesPerBlock - 1) {                   // the path goes on in the next workgroup
            if (left != kNoRow) {
                add_open(left, kWavesPerBlock);
                store_carry((int32_t)blockIdx.x);
            }
            if (lane == 0) a.carry_row[blockIdx.x] = left;
        }
    }
}

// Adds the carries of every split row to the part stored by the piece that finished the row, in order.
// One wave per carry; only the wave of a row's first carry does the work.  Lanes own the same column slices
// as in the main kernel, and several carries are in flight at once.
template <int VW, int NV>
__global__ __launch_bounds__(kBlock) void spmm_carry_kernel(const SpmmArgs a)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t item = uniform_i32((int32_t)(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)));
    if (item >= a.n_items) return;
    const int32_t r = uniform_i32(a.carry_row[item]);
    if (r < 0 || r >= a.n_rows) return;
    if (item > 0 && uniform_i32(a.carry_row[item - 1]) == r) return;
    int32_t last = item + 1;
    while (last < a.n_items && uniform_i32(a.carry_row[last]) == r) ++last;

    const bool last_ok = ((NV - 1) * kWave + lane) * VW < a.wdim;
    float sum[NV][VW];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < VW; ++k) sum[v][k] = 0.0f;
    constexpr int kAhead = 4;
    for (int32_t w0 = item; w0 < last; w0 += kAhead) {
        float c[kAhead][NV][VW];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int32_t w = w0 + u < last ? w0 + u : last - 1;
            const float *slot = a.carry + (int64_t)w * a.carry_ld;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                if (v < NV - 1 || last_ok) {
                    load_vec<VW>(slot + (v * kWave + lane) * VW, c[u][v]);
                } else {
#pragma unroll
                    for (int k = 0; k < VW; ++k) c[u][v][k] = 0.0f;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (w0 + u < last)
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int k = 0; k < VW; ++k) sum[v][k] += c[u][v][k];
    }
    float *o = a.out + (int64_t)r * a.ldo;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (v < NV - 1 || last_ok) {
            float cur[VW];
            load_vec<VW>(o + (v * kWave + lane) * VW, cur);
#pragma unroll
            for (int k = 0; k < VW; ++k) {
                cur[k] = cur[k] + sum[v][k];
                if (v == NV - 1 && (v * kWave + lane) * VW + k >= a.dim) cur[k] = 0.0f;      // row padding
            }
            store_vec<VW>(o + (v * kWave + lane) * VW, cur);
        }
    }
}

// Scratch of adaqp_spmm_csr_noalloc: one copy per GPU the library runs on, held until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress, never an address to pass to a kernel.
static __device__ __align__(256) unsigned char scratch[ADAQP_SPMM_NOALLOC_SCRATCH_BYTES];

// Geometry shared by the workspace query and the launch.
struct Geometry { int32_t n_items; int64_t carry_ld; int64_t bytes; int64_t carry_off; };

bool geometry(int64_t n_rows, int64_t nnz, int32_t dim, Geometry *g)
{
    const int64_t total = n_rows + nnz;
    if (total <= 0) { *g = Geometry{0, 0, 0, 0}; return true; }
    // path steps per wave: enough pieces to fill 256 CUs several times over, few enough that the search
    // and the carry are amortised
    int64_t per = 32;
    while (per < 512 && total / per > 65536) per *= 2;
    int64_t items = (total + per - 1) / per;
    if (items > (int64_t)1 << 30) return false;
    g->n_items = (int32_t)items;
    g->carry_ld = ((int64_t)dim + 31) / 32 * 32;
    g->carry_off = (items * 4 + 255) / 256 * 256;
    g->bytes = g->carry_off + (items * g->carry_ld * 4 + 255) / 256 * 256;
    return true;
}

// Pieces of the merge-path kernel for rows that share lines: of at least 64 or 128 steps, or n_items.  Nearly every piece leaves a row
// to the next, so short ones are held up by searches and carries once 6 000 of them fill the chip (send, receive and sums together,
// pieces of 32 steps / as here: 8 000 rows of 30 entries, 72 columns 45.9 / 36.6 us; 60 000 of 16, 72 columns 107 / 85, 130 columns
// 126 / 110; 30 000 of 55, 72 columns 165 / 122; 90 000 of 5, 72 columns 70.8 / 71.2).  Wide rows stay as they are: 64 steps gave 1.02
// at 301 and 470 columns, 128 0.94 to 1.05.  So do whole lines (90 000 rows of 5, 160 columns: 0.945).
constexpr int32_t kNarrow = 160;            // columns

int32_t longer_pieces(int64_t total, int32_t dim, int32_t n_items)
{
    int64_t per = 32;
    while (per < 128 && total / per > 6000) per *= 2;
    const int64_t items = (total + per - 1) / per;
    return dim <= kNarrow && items < n_items ? (int32_t)items : n_items;
}

template <int VW, int NV>
hipError_t launch_merge(const SpmmArgs &a, bool chains, bool joins, hipStream_t st)
{
    constexpr int U = NV >= 4 ? 4 : (NV >= 2 ? 8 : 16);
    constexpr bool kMay = (NV - 1) * kWave * VW < kNarrow;      // some row with so many vectors is narrow
    auto kernel_of = [&](auto with_chains, auto with_joins) {
        constexpr bool kChains = decltype(with_chains)::value, kJoins = decltype(with_joins)::value;
        return a.p.slot_of_row ? spmm_merge_kernel<VW, NV, U, true, kChains, kJoins> : spmm_merge_kernel<VW, NV, U, false, kChains, kJoins>;
    };
    joins = joins && VW * NV <= kJoinFloats;
    auto kernel = kernel_of(std::false_type(), std::false_type());
    if constexpr (kMay)
        if (chains) kernel = kernel_of(std::true_type(), std::false_type());
    if constexpr (VW * NV <= kJoinFloats) {
        if (joins) kernel = kernel_of(std::false_type(), std::true_type());
        if constexpr (kMay)
            if (joins && chains) kernel = kernel_of(std::true_type(), std::true_type());
    }
    const dim3 grid((unsigned)((a.n_items + kWavesPerBlock - 1) / kWavesPerBlock));
    hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, st, a);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    SpmmArgs carries = a;
    if (joins) carries.n_items = (int32_t)grid.x;               // one of a workgroup
    hipLaunchKernelGGL((spmm_carry_kernel<VW, NV>), dim3((carries.n_items + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlock), 0, st, carries);
    return hipGetLastError();
}

template <int VW>
hipError_t launch_merge_nv(const SpmmArgs &a, int nv, bool chains, bool joins, hipStream_t st)
{
    switch (nv) {
        case 1: return launch_merge<VW, 1>(a, chains, joins, st);
        case 2: return launch_merge<VW, 2>(a, chains, joins, st);
        case 3: return launch_merge<VW, 3>(a, chains, joins, st);
        case 4: return launch_merge<VW, 4>(a, chains, joins, st);
        case 5: return launch_merge<VW, 5>(a, chains, joins, st);
        case 6: return launch_merge<VW, 6>(a, chains, joins, st);
        case 7: return launch_merge<VW, 7>(a, chains, joins, st);
        case 8: return launch_merge<VW, 8>(a, chains, joins, st);
        default: return hipErrorInvalidValue;
    }
}

template <int VW>
hipError_t launch_carry_nv(const SpmmArgs &a, int nv, hipStream_t st)
{
    const dim3 grid((unsigned)((a.n_items + kWavesPerBlock - 1) / kWavesPerBlock));
    switch (nv) {
#define ADAQP_CASE(N) case N: hipLaunchKernelGGL((spmm_carry_kernel<VW, N>), grid, dim3(kBlock), 0, st, a); break;
        ADAQP_CASE(1) ADAQP_CASE(2) ADAQP_CASE(3) ADAQP_CASE(4)
        ADAQP_CASE(5) ADAQP_CASE(6) ADAQP_CASE(7) ADAQP_CASE(8)
#undef ADAQP_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace adaqp

using namespace adaqp;

extern "C" int adaqp_spmm_workspace_bytes(int64_t n_rows, int64_t nnz, int32_t dim, int64_t *bytes_out)
{
    if (!bytes_out || n_rows < 0 || nnz < 0 || dim <= 0) return ADAQP_EINVAL;
    Geometry g;
    if (!geometry(n_rows, nnz, dim, &g)) return ADAQP_ESIZE;
    *bytes_out = g.bytes;
    return ADAQP_OK;
}

extern "C" int adaqp_spmm_csr(const int64_t *rowptr_dev, const int32_t *col_dev, const float *val_dev,
                              int64_t nnz, int64_t row_begin, int64_t row_end, int64_t nnz_range,
                              const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
                              float *out_dev, int64_t ldo, void *workspace_dev, int64_t workspace_bytes,
                              void *stream)
{
    return adaqp_spmm_csr_packed(rowptr_dev, col_dev, val_dev, nnz, row_begin, row_end, nnz_range, H_dev, n_cols, ldh,
                                 dim, out_dev, ldo, nullptr, nullptr, 0, nullptr, nullptr, nullptr, 0, workspace_dev,
                                 workspace_bytes, stream);
}

extern "C" int adaqp_spmm_csr_packed(const int64_t *rowptr_dev, const int32_t *col_dev, const float *val_dev,
                                     int64_t nnz, int64_t row_begin, int64_t row_end, int64_t nnz_range,
                                     const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
                                     float *out_dev, int64_t ldo,
                                     const int32_t *slot_of_row_dev, const uint8_t *packed_dev, int64_t packed_bytes,
                                     const float *params_dev, const uint8_t *bits_dev, const int64_t *row_offset_dev,
                                     int64_t n_slots,
                                     void *workspace_dev, int64_t workspace_bytes, void *stream)
{
    return spmm_rows(rowptr_dev, col_dev, val_dev, nnz, row_begin, row_end, nnz_range, H_dev, n_cols, ldh, dim, out_dev, ldo,
                     slot_of_row_dev, packed_dev, packed_bytes, params_dev, bits_dev, row_offset_dev, n_slots,
                     workspace_dev, workspace_bytes, stream, false);
}

int adaqp::spmm_rows(const int64_t *rowptr_dev, const int32_t *col_dev, const float *val_dev,
                     int64_t nnz, int64_t row_begin, int64_t row_end, int64_t nnz_range,
                     const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
                     float *out_dev, int64_t ldo,
                     const int32_t *slot_of_row_dev, const uint8_t *packed_dev, int64_t packed_bytes,
                     const float *params_dev, const uint8_t *bits_dev, const int64_t *row_offset_dev,
                     int64_t n_slots,
                     void *workspace_dev, int64_t workspace_bytes, void *stream, bool skewed_columns)
{
    if (slot_of_row_dev) {
        if (!packed_dev || !params_dev || !bits_dev || !row_offset_dev || packed_bytes < 4 || n_slots <= 0)
            return ADAQP_EINVAL;
        if (!aligned_to(slot_of_row_dev, 4) || !aligned_to(packed_dev, 4) || !aligned_to(params_dev, 8) ||
            !aligned_to(row_offset_dev, 8))
            return ADAQP_EINVAL;
    }
    if (row_begin < 0 || row_end < row_begin || nnz < 0 || dim <= 0 || ldh < dim || ldo < dim || n_cols < 0)
        return ADAQP_EINVAL;
    const int64_t n_rows = row_end - row_begin;
    if (n_rows == 0) return ADAQP_OK;
    if (!rowptr_dev || !out_dev) return ADAQP_EINVAL;
    if (nnz > 0 && (!col_dev || !val_dev || !H_dev || n_cols == 0)) return ADAQP_EINVAL;
    if (n_rows > INT32_MAX - 1) return ADAQP_ESIZE;
    if (!aligned_to(rowptr_dev, 8) || !aligned_to(col_dev, 4) || !aligned_to(val_dev, 4) ||
        !aligned_to(H_dev, 4) || !aligned_to(out_dev, 4))
        return ADAQP_EINVAL;
    if (nnz_range < 0 || nnz_range > nnz) nnz_range = nnz;

    Geometry g;
    if (!geometry(n_rows, nnz_range, dim, &g)) return ADAQP_ESIZE;
    if (g.bytes > 0 && (!workspace_dev || !aligned_to(workspace_dev, 256))) return ADAQP_EINVAL;
    if (workspace_bytes < g.bytes) return ADAQP_ESIZE;

    // vector width: every row start of H and out and of the carry slots must be naturally aligned, and a
    // vector must not spill past dim - unless both matrices are line-padded (rows start on 128-byte lines,
    // pitch a whole number of lines): then rows are read and written in whole lines, padding written as zero
    const bool whole_lines = ldh % 32 == 0 && ldo % 32 == 0 && aligned_to(H_dev, 128) && aligned_to(out_dev, 128);
    int vw = 1;
    if (whole_lines) vw = 4;
    else if (dim % 4 == 0 && ldh % 4 == 0 && ldo % 4 == 0 && aligned_to(H_dev, 16) && aligned_to(out_dev, 16)) vw = 4;
    else if (dim % 2 == 0 && ldh % 2 == 0 && ldo % 2 == 0 && aligned_to(H_dev, 8) && aligned_to(out_dev, 8)) vw = 2;

    hipStream_t st = (hipStream_t)stream;
    const int32_t chunk_cap = kWave * vw * 8;               // columns one launch covers (NV <= 8)
    for (int32_t c0 = 0; c0 < dim; c0 += chunk_cap) {
        const int32_t cdim = dim - c0 < chunk_cap ? dim - c0 : chunk_cap;
        SpmmArgs a;
        a.rowptr = rowptr_dev + row_begin;
        a.col = col_dev;
        a.val = val_dev;
        a.nnz = nnz;
        a.n_rows = (int32_t)n_rows;
        a.H = H_dev + c0;
        a.n_cols = n_cols;
        a.ldh = ldh;
        a.dim = cdim;
        a.wdim = whole_lines ? (cdim + 31) / 32 * 32 : cdim;
        a.out = out_dev + row_begin * ldo + c0;
        a.ldo = ldo;
        a.carry_row = reinterpret_cast<int32_t *>(workspace_dev);
        a.carry = reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(workspace_dev) + g.carry_off);
        a.carry_ld = g.carry_ld;
        a.n_items = g.n_items;
        a.p.slot_of_row = slot_of_row_dev;
        a.p.col0 = c0;
        a.p.full_dim = dim;
        a.p.packed = packed_dev;
        a.p.packed_bytes = packed_bytes;
        a.p.params = params_dev;
        a.p.bits = bits_dev;
        a.p.row_offset = row_offset_dev;
        a.p.n_slots = n_slots;
        const int nv = (a.wdim + kWave * vw - 1) / (kWave * vw);
        hipError_t err;
        const SlicedCut cut = plan_sliced(a, nnz_range, whole_lines, skewed_columns);
        if (cut.lines > 0) {
            err = launch_sliced(a, cut, nnz_range, whole_lines, st, &a.n_items);
            if (err == hipSuccess)
                err = vw == 4 ? launch_carry_nv<4>(a, nv, st)
                              : (vw == 2 ? launch_carry_nv<2>(a, nv, st) : launch_carry_nv<1>(a, nv, st));
        } else {
            if (!whole_lines) a.n_items = longer_pieces(n_rows + nnz_range, dim, g.n_items);
            const bool chains = a.n_items < g.n_items, joins = merge_joins(n_rows, nnz_range, a.n_items, dim);
            err = vw == 4 ? launch_merge_nv<4>(a, nv, chains, joins, st)
                          : (vw == 2 ? launch_merge_nv<2>(a, nv, chains, joins, st) : launch_merge_nv<1>(a, nv, chains, joins, st));
        }
        ADAQP_HIP_TRY(err);
    }
    return ADAQP_OK;
}

// ---- segments: the sliced kernel over the entries in tile order ----------------------------------------------------------

namespace {

constexpr int kSegments = ADAQP_SPMM_SEGMENTS;
static_assert(kSegments == ADAQP_SPMM_TILES, "a row has a segment per tile at most");
constexpr int kUpdateLanes = 32;

// Workgroups per slice.  The fewer entries are under way at a time, the fewer groups of tiles an L2 has to hold, but a share is a
// search and an empty ring: shares of about 1 100 entries (2.5 M entries, 602 columns: 256 workgroups 0.44 ms, 512 0.41, 1 024 0.42, 2 048
// 0.54; 3.5 M: 0.70, 0.57, 0.58, 0.66), no more than 1 024 workgroups (15 M entries, 256 columns: 512 0.78, 1 024 0.75, 2 048 0.79).
int64_t segment_blocks(int64_t n_seg, int64_t n_entries)
{
    const int64_t wanted = std::min<int64_t>(std::max<int64_t>(n_entries / 4500, 256), 1024);
    return std::max<int64_t>(std::min(wanted, (n_entries + 8 * n_seg) / 1024), 1);
}

struct SegmentGeometry { int64_t n_items, wdim, carry_row_off, carry_off, bytes; };

SegmentGeometry segment_geometry(int64_t n_seg, int64_t n_entries, int32_t dim)
{
    SegmentGeometry g;
    g.wdim = ((int64_t)dim + 31) / 32 * 32;
    g.n_items = segment_blocks(n_seg, n_entries) * kWavesPerBlock;
    g.carry_row_off = (n_seg * g.wdim * 4 + 255) / 256 * 256;
    g.carry_off = g.carry_row_off + (g.n_items * 4 + 255) / 256 * 256;
    g.bytes = g.carry_off + (g.n_items * g.wdim * 4 + 255) / 256 * 256;
    return g;
}

constexpr int32_t kGroupCols = 12288;

// First tile of each group, and behind the last one; 0 groups: bounds that descend.
int segment_groups(const int32_t *col_bounds, int (&first_tile)[ADAQP_SPMM_TILES + 1])
{
    int n_groups = 0;
    for (int t = 0; t < ADAQP_SPMM_TILES; ++t) {
        if (col_bounds[t + 1] < col_bounds[t]) return 0;
        if (n_groups == 0 || col_bounds[t + 1] - col_bounds[first_tile[n_groups - 1]] > kGroupCols) first_tile[n_groups++] = t;
    }
    first_tile[n_groups] = ADAQP_SPMM_TILES;
    return n_groups;
}

// A wave per segment.
__global__ __launch_bounds__(kBlock) void segments_fill_kernel(const int64_t *ptr, const int64_t *src, int64_t n_seg, int64_t n_entries,
                                                               const int32_t *col, const float *val, int64_t nnz, int32_t *col_out,
                                                               float *val_out)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t s = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave; s < n_seg; s += waves) {
        const int64_t to = clamp64(ptr[s], 0, n_entries), n = clamp64(ptr[s + 1], to, n_entries) - to;
        const int64_t from = src[s];
        for (int64_t i = lane; i < n; i += kWave) {
            const bool in = from >= 0 && from + i < nnz;
            col_out[to + i] = in ? col[from + i] : -1;
            val_out[to + i] = in ? val[from + i] : 0.0f;
        }
    }
}

// val_out where it is not what val says.  Bound by the reads of both streams and by their latency where segments are short: 27.8 M entries
// in segments of 63 0.104 ms (2.1 TB/s), 7.7 M in segments of 20 0.051.  Half a wave per segment: of 8, 16, 32 and 64 lanes segments of
// 20 take 33, 28, 30 and 43 us (4.6 M entries), of 40 16, 13, 12 and 14 (2.5 M), of 63 84, 65, 52 and 50 (13.3 M).
__global__ __launch_bounds__(kBlock) void segments_update_kernel(const int64_t *ptr, const int64_t *src, int64_t n_seg, int64_t n_entries,
                                                                 const uint32_t *val, int64_t nnz, uint32_t *val_out)
{
    const int lane = threadIdx.x & (kUpdateLanes - 1);
    const int64_t groups = (int64_t)gridDim.x * (kBlock / kUpdateLanes);
    for (int64_t s = (int64_t)blockIdx.x * (kBlock / kUpdateLanes) + threadIdx.x / kUpdateLanes; s < n_seg; s += groups) {
        const int64_t to = clamp64(ptr[s], 0, n_entries), n = clamp64(ptr[s + 1], to, n_entries) - to;
        const int64_t from = src[s];
        for (int64_t i = lane; i < n; i += kUpdateLanes) {
            const uint32_t now = from >= 0 && from + i < nnz ? val[from + i] : 0;
            if (now != val_out[to + i]) val_out[to + i] = now;
        }
    }
}

// out[r] = sum of the row's segments in group order; whole lines, row padding zero.  A wave per row: all segments of a strip of 256
// columns in flight together.
__global__ __launch_bounds__(kBlock) void segments_sum_kernel(const int32_t *of_row, int64_t n_rows, int64_t n_seg, const float *partial,
                                                              int32_t dim, int32_t wdim, float *out, int64_t ldo)
{
    typedef float float4_t __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
    if (r >= n_rows) return;
    int32_t seg[kSegments];
#pragma unroll
    for (int q = 0; q < kSegments; ++q) seg[q] = uniform_i32(of_row[r * kSegments + q]);
    if (seg[0] < -1) return;                                // a row struck from the table: someone else's to write
    for (int32_t c = lane * 4; c < wdim; c += kWave * 4) {
        float4_t x[kSegments];
#pragma unroll
        for (int q = 0; q < kSegments; ++q) {
            x[q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if (seg[q] >= 0 && seg[q] < n_seg)
                x[q] = __builtin_nontemporal_load(reinterpret_cast<const float4_t *>(partial + (int64_t)seg[q] * wdim + c));
        }
        float4_t sum = x[0];
#pragma unroll
        for (int q = 1; q < kSegments; ++q) sum += x[q];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k >= dim) sum[k] = 0.0f;
        __builtin_nontemporal_store(sum, reinterpret_cast<float4_t *>(out + r * ldo + c));
    }
}

}  // namespace

extern "C" int adaqp_plan_spmm_segments(const int64_t *rowptr_host, int64_t row_begin, int64_t row_end, const int32_t *col_bounds_host,
                                        const int32_t *tile_off_host, int64_t *sizes_inout, int64_t *ptr_out, int64_t *src_out,
                                        int32_t *of_row_out)
{
    constexpr int T = ADAQP_SPMM_TILES;
    if (row_begin < 0 || row_end < row_begin || !rowptr_host || !col_bounds_host || !sizes_inout) return ADAQP_EINVAL;
    const int64_t n_rows = row_end - row_begin;
    if (n_rows > 0 && !tile_off_host) return ADAQP_EINVAL;
    const bool fill = ptr_out != nullptr;
    if (fill && (!src_out || (n_rows > 0 && !of_row_out))) return ADAQP_EINVAL;
    // Groups of tiles (segment_groups): an L2 of 4 MB holds two lines of 16 384 columns.  Sums included, 12.7 M entries in 58 000 columns, 256 columns of
    // H: groups of 7 000 columns 0.64 ms, 14 000 0.65, 21 000 0.70, 29 000 0.72; 15 M in 98 000 columns: 13 000 0.75, 24 000 0.77, 32 000
    // 0.81.  Smaller graphs with short segments: 2.5 M entries in 58 000 columns, 602 columns of H 0.41, 0.42, 0.43, 0.47.
    int first_tile[T + 1];
    const int n_groups = segment_groups(col_bounds_host, first_tile);
    if (n_groups == 0) return ADAQP_EINVAL;
    int64_t n_seg = 0, n_entries = 0;
    for (int g = 0; g < n_groups; ++g)
        for (int64_t r = 0; r < n_rows; ++r) {
            const int32_t *off = tile_off_host + r * (T + 1);
            const int64_t first = rowptr_host[row_begin + r], degree = rowptr_host[row_begin + r + 1] - first;
            if (off[0] < 0) {
                if (fill) of_row_out[r * kSegments + g] = g == 0 ? -2 : -1;
                continue;
            }
            const int32_t a = off[first_tile[g]], b = off[first_tile[g + 1]];
            if (a < 0 || b < a || b > degree || (g == 0 && off[0] != 0) || (g + 1 == n_groups && off[T] != degree)) return ADAQP_EINVAL;
            if (fill) of_row_out[r * kSegments + g] = b > a ? (int32_t)n_seg : -1;
            if (b == a) continue;
            if (fill) {
                if (n_seg >= sizes_inout[0]) return ADAQP_EINVAL;
                ptr_out[n_seg] = n_entries;
                src_out[n_seg] = first + a;
            }
            ++n_seg;
            n_entries += b - a;
        }
    if (n_seg > INT32_MAX - 1024) return ADAQP_ESIZE;
    if (!fill) {
        sizes_inout[0] = n_seg;
        sizes_inout[1] = n_entries;
        return ADAQP_OK;
    }
    if (n_seg != sizes_inout[0] || n_entries != sizes_inout[1]) return ADAQP_EINVAL;
    ptr_out[n_seg] = n_entries;
    for (int g = n_groups; g < kSegments; ++g)
        for (int64_t r = 0; r < n_rows; ++r) of_row_out[r * kSegments + g] = -1;
    return ADAQP_OK;
}

// Two lines where an L2 of 4 MB holds them of a good part of a group, else one: 12 300 columns per group, 28 M entries, 256 columns of H 1.46
// and 1.19 ms with one and two; 57 000 columns per group, 7.7 M entries 0.75 and 0.83; 400 steps, one against two: 16 000 to 25 000 columns
// 1.01, 25 000 to 38 000 0.97, more 0.93.
extern "C" int32_t adaqp_spmm_segments_lines(const int32_t *col_bounds_host)
{
    int first_tile[ADAQP_SPMM_TILES + 1];
    const int n_groups = col_bounds_host ? segment_groups(col_bounds_host, first_tile) : 0;
    int32_t widest = 0;
    for (int g = 0; g < n_groups; ++g) widest = std::max(widest, col_bounds_host[first_tile[g + 1]] - col_bounds_host[first_tile[g]]);
    return widest > 20480 ? 1 : 2;
}

// What segments save is what the sliced kernel misses in its L2s: entries of rows that are cut up (shorter ones lie whole in one group and
// find no more there than before), but for those whose columns are the most popular ones.  What they cost is the walk over all
// entries, and a partial row and its sum per row.  1 370 steps of 5 000 to 300 000 rows, 20 to 500 entries per row, 64 to
// 602 columns of H, Zipf and log-normal rows, both directions, timed with and without; with the weights below none loses more than 8 %.
// Geometric mean against no segments forward 1.117 (the better of both each time 1.120), backward 1.043 (1.049); segments from
// a mean of 128 entries per row on 1.055 and 0.954 (power-law degrees there 0.34-0.75: a few columns hold most of the
// entries).  150 000 rows, 256 columns: 48 entries per row 898 -> 675 us, 100 entries 1 808 -> 1 109 us.
extern "C" int adaqp_spmm_segments_gain(const int64_t *rowptr_host, const int32_t *col_host, int64_t row_begin, int64_t row_end, int64_t n_cols,
                                        int32_t dim, int32_t transposed, double *gain_out)
{
    if (!rowptr_host || !gain_out || row_begin < 0 || row_end < row_begin || n_cols < 0 || n_cols > INT32_MAX || dim <= 0) return ADAQP_EINVAL;
    constexpr int64_t kPopular = 4096;          // columns that stay in an L2 beside everything else
    constexpr int64_t kSample = 1 << 22;        // entries looked at for that
    const int64_t first = rowptr_host[row_begin], last = rowptr_host[row_end], block_row = adaqp_spmm_blocks_min_row(n_cols);
    if (first < 0 || last < first) return ADAQP_EINVAL;
    const double lines = (double)(((int64_t)dim + 31) / 32);
    double cut = 0.0, dense = 0.0;              // entries of rows that are cut up, of rows for the matrix cores
    int64_t n_dense = 0;
    for (int64_t r = row_begin; r < row_end; ++r) {
        const int64_t degree = rowptr_host[r + 1] - rowptr_host[r];
        if (degree < 0) return ADAQP_EINVAL;
        if (degree >= ADAQP_SPMM_TILED_SHORT_ROW) cut += (double)degree;
        if (degree >= block_row) {
            dense += (double)degree;
            ++n_dense;
        }
    }
    const bool asked_for = adaqp_spmm_tiled_pays(row_end - row_begin, last - first) != 0;
    if (last > first && !col_host) return ADAQP_EINVAL;
    // every range, also one that cannot gain: it would be tiled with the other ranges of its step
    for (int64_t r = row_begin; r < row_end; ++r) {
        int32_t before = -1;
        for (int64_t j = rowptr_host[r]; j < rowptr_host[r + 1]; ++j) {
            const int32_t c = col_host[j];
            if (c <= before || c >= n_cols) {
                *gain_out = -INFINITY;
                return asked_for ? ADAQP_EINVAL : ADAQP_OK;
            }
            before = c;
        }
    }
    if (!adaqp_spmm_blocks_pay(n_dense, n_cols, 32)) dense = 0.0;
    const double entries = (double)(last - first), rows = (double)(row_end - row_begin);
    *gain_out = (transposed ? 0.0 : blocks_gain(lines, dense)) - segments_cost(transposed != 0, lines, entries, rows);
    if (!asked_for && cut * lines + *gain_out <= 0.0) return ADAQP_OK;         // whatever the columns are
    std::vector<int32_t> uses;
    try {
        uses.resize((size_t)n_cols, 0);
    } catch (const std::bad_alloc &) {          // nothing may be thrown through a C entry; the plan would have no room either
        *gain_out = -INFINITY;
        return ADAQP_OK;
    }
    const int64_t stride = std::max<int64_t>((last - first) / kSample, 1);
    int64_t seen = 0;
    for (int64_t j = first; j < last; j += stride, ++seen) ++uses[(size_t)col_host[j]];
    if (n_cols > kPopular) std::nth_element(uses.begin(), uses.begin() + kPopular, uses.end(), std::greater<int32_t>());
    const int64_t popular = std::accumulate(uses.begin(), uses.begin() + std::min(kPopular, n_cols), (int64_t)0);
    if (seen > 0) *gain_out += cut * lines * (1.0 - (double)popular / (double)seen);
    return ADAQP_OK;
}

extern "C" int adaqp_fill_spmm_segments(const adaqp_spmm_segments *p, const int32_t *col_dev, const float *val_dev, int64_t nnz, void *stream)
{
    if (!p || p->n_seg < 0 || p->n_entries < 0 || nnz < 0) return ADAQP_EINVAL;
    if (p->n_seg == 0 || p->n_entries == 0) return ADAQP_OK;
    if (!p->ptr_dev || !p->src_dev || !p->col_dev || !p->val_dev || (nnz > 0 && (!col_dev || !val_dev))) return ADAQP_EINVAL;
    hipLaunchKernelGGL(segments_fill_kernel, dim3((unsigned)std::min<int64_t>((p->n_seg + kWavesPerBlock - 1) / kWavesPerBlock, 65536)), dim3(kBlock),
                       0, (hipStream_t)stream, p->ptr_dev, p->src_dev, p->n_seg, p->n_entries, col_dev, val_dev, nnz, p->col_dev, p->val_dev);
    ADAQP_HIP_TRY(hipGetLastError());
    return ADAQP_OK;
}

extern "C" int adaqp_update_spmm_segments(const adaqp_spmm_segments *p, const float *val_dev, int64_t nnz, void *stream)
{
    if (!p || p->n_seg < 0 || p->n_entries < 0 || nnz < 0) return ADAQP_EINVAL;
    if (p->n_seg == 0 || p->n_entries == 0) return ADAQP_OK;
    if (!p->ptr_dev || !p->src_dev || !p->val_dev || (nnz > 0 && !val_dev)) return ADAQP_EINVAL;
    constexpr int64_t kPerBlock = kBlock / kUpdateLanes;
    hipLaunchKernelGGL(segments_update_kernel, dim3((unsigned)std::min<int64_t>((p->n_seg + kPerBlock - 1) / kPerBlock, 65536)), dim3(kBlock), 0,
                       (hipStream_t)stream, p->ptr_dev, p->src_dev, p->n_seg, p->n_entries, reinterpret_cast<const uint32_t *>(val_dev), nnz,
                       reinterpret_cast<uint32_t *>(p->val_dev));
    ADAQP_HIP_TRY(hipGetLastError());
    return ADAQP_OK;
}

extern "C" int adaqp_spmm_segments_workspace_bytes(int64_t n_seg, int64_t n_entries, int32_t dim, int64_t *bytes_out)
{
    if (!bytes_out || n_seg < 0 || n_entries < 0 || dim <= 0) return ADAQP_EINVAL;
    if (n_seg > INT32_MAX - 1024) return ADAQP_ESIZE;
    *bytes_out = n_seg == 0 ? 0 : segment_geometry(n_seg, n_entries, dim).bytes;
    return ADAQP_OK;
}

int adaqp::check_segments_call(const adaqp_spmm_segments *p, const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim, const float *out_dev,
                               int64_t ldo)
{
    if (!p || p->n_seg < 0 || p->n_entries < 0 || p->n_rows < 0 || n_cols < 0 || dim <= 0 || ldh < dim || ldo < dim) return ADAQP_EINVAL;
    if (p->n_seg == 0 || p->n_rows == 0) return ADAQP_OK;
    if (!p->ptr_dev || !p->of_row_dev || !p->col_dev || !p->val_dev || !H_dev || !out_dev || n_cols == 0 || p->n_entries == 0) return ADAQP_EINVAL;
    if (!aligned_to(p->ptr_dev, 8) || !aligned_to(p->of_row_dev, 4) || !aligned_to(p->col_dev, 4) || !aligned_to(p->val_dev, 4)) return ADAQP_EINVAL;
    if (ldh % 32 != 0 || ldo % 32 != 0 || !aligned_to(H_dev, 128) || !aligned_to(out_dev, 128)) return ADAQP_EINVAL;
    if (p->pieces.n_pieces != 0) {
        const int rc = check_pieces(&p->pieces, p->n_seg);
        if (rc != ADAQP_OK) return rc;
    }
    if (p->n_seg > INT32_MAX - 1024 || p->n_rows > INT32_MAX - 1 || !sliced_takes(p->n_seg, p->n_entries, n_cols, ldh, false, 0, dim)) return ADAQP_ESIZE;
    return ADAQP_OK;
}

extern "C" int adaqp_spmm_csr_segments(const adaqp_spmm_segments *p, const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
                                       float *out_dev, int64_t ldo, void *workspace_dev, int64_t workspace_bytes, void *stream)
{
    const int rc = check_segments_call(p, H_dev, n_cols, ldh, dim, out_dev, ldo);
    if (rc != ADAQP_OK || p->n_seg == 0 || p->n_rows == 0) return rc;
    if (p->pieces.n_pieces > 0) {
        int64_t need = 0;
        ADAQP_TRY(adaqp_spmm_pieces_workspace_bytes(p->pieces.n_partials, dim, &need));
        if (need > 0 && (!workspace_dev || !aligned_to(workspace_dev, 256))) return ADAQP_EINVAL;
        if (workspace_bytes < need) return ADAQP_ESIZE;
        PieceArgs a = {};
        a.ptr = p->ptr_dev;
        a.col = p->col_dev;
        a.val = p->val_dev;
        a.n_entries = p->n_entries;
        a.n_seg = (int32_t)p->n_seg;
        a.H = H_dev;
        a.n_cols = n_cols;
        a.ldh = ldh;
        a.dim = dim;
        a.out = out_dev;
        a.ldo = ldo;
        a.n_rows = (int32_t)p->n_rows;
        a.partial = reinterpret_cast<float *>(workspace_dev);
        return launch_pieces(&p->pieces, a, (hipStream_t)stream);
    }
    const SegmentGeometry g = segment_geometry(p->n_seg, p->n_entries, dim);
    if (!workspace_dev || !aligned_to(workspace_dev, 256)) return ADAQP_EINVAL;
    if (workspace_bytes < g.bytes) return ADAQP_ESIZE;

    char *ws = static_cast<char *>(workspace_dev);
    float *partial = reinterpret_cast<float *>(ws);
    hipStream_t st = (hipStream_t)stream;
    constexpr int32_t kCap = kWave * 4 * 8;                 // columns one launch covers
    for (int32_t c0 = 0; c0 < dim; c0 += kCap) {
        SpmmArgs a = {};
        a.rowptr = p->ptr_dev;
        a.col = p->col_dev;
        a.val = p->val_dev;
        a.nnz = p->n_entries;
        a.n_rows = (int32_t)p->n_seg;
        a.H = H_dev + c0;
        a.n_cols = n_cols;
        a.ldh = ldh;
        a.dim = std::min(dim - c0, kCap);
        a.wdim = (a.dim + 31) / 32 * 32;
        a.out = partial + c0;
        a.ldo = g.wdim;
        a.carry_row = reinterpret_cast<int32_t *>(ws + g.carry_row_off);
        a.carry = reinterpret_cast<float *>(ws + g.carry_off);
        a.carry_ld = g.wdim;
        a.n_items = (int32_t)g.n_items;
        a.p.full_dim = dim;
        // two lines per slice (15 M entries, 98 000 columns: one line 0.80 ms, two 0.75, four 0.81)
        const SlicedCut cut = {a.wdim > 32 ? 2 : 1, 0, segment_blocks(p->n_seg, p->n_entries)};
        ADAQP_HIP_TRY(launch_sliced(a, cut, p->n_entries, true, st, &a.n_items));
        ADAQP_HIP_TRY(launch_carry_nv<4>(a, (a.wdim + kWave * 4 - 1) / (kWave * 4), st));
    }
    constexpr int64_t kMostRows = (int64_t)1 << 24;         // of a launch, which has fewer than 2^32 threads (a loop in the kernel: 306 000
                                                            // rows, 256 columns 1.036 -> 1.065 ms for the whole step)
    for (int64_t r0 = 0; r0 < p->n_rows; r0 += kMostRows) {
        const int64_t rows = std::min(p->n_rows - r0, kMostRows);
        hipLaunchKernelGGL(segments_sum_kernel, dim3((unsigned)((rows + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(kBlock), 0, st,
                           p->of_row_dev + r0 * kSegments, rows, p->n_seg, partial, dim, (int32_t)g.wdim, out_dev + r0 * ldo, ldo);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    return ADAQP_OK;
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];      // device address of `scratch` on each GPU, looked up once per GPU

// Address of the current device's copy of `scratch`.  The first call on a device asks the runtime for it (which
// may load the code object); later calls only read the table.
int scratch_of_current_device(void **ptr_out)
{
    int dev = -1;
    ADAQP_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return ADAQP_ESIZE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        ADAQP_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return note_hip_error(hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = p;
    }
    *ptr_out = g_scratch_ptr[dev];
    return ADAQP_OK;
}

}  // namespace

extern "C" int adaqp_spmm_csr_noalloc(const int64_t *rowptr_dev, const int32_t *col_dev, const float *val_dev,
                                      int64_t nnz, int64_t row_begin, int64_t row_end, int64_t nnz_range,
                                      const float *H_dev, int64_t n_cols, int64_t ldh, int32_t dim,
                                      float *out_dev, int64_t ldo, void *stream)
{
    // the same checks, in the same order, as adaqp_spmm_csr makes before it looks at its workspace
    if (row_begin < 0 || row_end < row_begin || nnz < 0 || dim <= 0 || ldh < dim || ldo < dim || n_cols < 0)
        return ADAQP_EINVAL;
    const int64_t n_rows = row_end - row_begin;
    if (n_rows == 0) return ADAQP_OK;
    if (!rowptr_dev || !out_dev) return ADAQP_EINVAL;
    if (nnz > 0 && (!col_dev || !val_dev || !H_dev || n_cols == 0)) return ADAQP_EINVAL;
    if (n_rows > INT32_MAX - 1) return ADAQP_ESIZE;
    if (!aligned_to(rowptr_dev, 8) || !aligned_to(col_dev, 4) || !aligned_to(val_dev, 4) ||
        !aligned_to(H_dev, 4) || !aligned_to(out_dev, 4))
        return ADAQP_EINVAL;
    Geometry g;
    if (!geometry(n_rows, (nnz_range < 0 || nnz_range > nnz) ? nnz : nnz_range, dim, &g)) return ADAQP_ESIZE;
    if (g.bytes > (int64_t)ADAQP_SPMM_NOALLOC_SCRATCH_BYTES) return ADAQP_ESIZE;     // beyond the built-in scratch
    void *ptr = nullptr;
    const int rc = scratch_of_current_device(&ptr);
    if (rc != ADAQP_OK) return rc;
    return adaqp_spmm_csr(rowptr_dev, col_dev, val_dev, nnz, row_begin, row_end, nnz_range, H_dev, n_cols, ldh, dim,
                          out_dev, ldo, ptr, (int64_t)ADAQP_SPMM_NOALLOC_SCRATCH_BYTES, stream);
}
