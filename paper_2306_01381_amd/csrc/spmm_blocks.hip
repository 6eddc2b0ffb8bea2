// Neighbour aggregation (Sec. 2.1 Eq. 3) for rows that list a good part of all columns, as a dense product on the bf16
// matrix cores with fp32 operands split in three.
//
// Where rows have thousands of entries (Sec. 5: mean degree near 500 with a heavy tail) 128 of them together reference nearly
// every column, each 20 to 60 times.  The host plan takes such rows 128 at a time, longest first: the sorted distinct columns of
// the block and a dense [columns][128] table of fp32 coefficients.  out[block rows] = table^T x H[columns].
//
// fp32 to the matrix cores: the bf16 instructions run at 16 times the rate of the fp32 ones.  A value is hi + mid + lo, three
// bf16, exactly, each rounded to nearest, so that mid is at most 2^-8 of it and lo 2^-17.  A product takes six of the nine partial
// products; mid x lo, lo x mid and lo x lo are left out, at most 2^-25, 2^-25 and 2^-34 of the product and together less than
// 2^-24, half a unit in the last place (over all pairs of mantissas; with hi cut off instead of rounded 3.96 * 2^-24).
// hi x hi goes into sums of its own: the instruction drops the bits of a product that lie far below the accumulator, and next
// to a long sum the small products would lose theirs (one set of sums: relative error 4.6e-7 on rows of 6 000 entries and more
// of normal features, 1.7e-7 on non-negative ones; two sets 1.3e-7 and 5.0e-8; fp32 instructions 2.9e-7 and 5.3e-8).
//
// A workgroup takes one piece (a block's columns in one interval of the columns of H) x 128 feature columns.  Per step of 32
// of the block's columns each of its four waves loads the rows of H for 32 feature columns, splits them (3.5 instructions per
// value) and leaves them in LDS as matrix operands; then each takes 32 of the block's rows, splits its coefficients and
// multiplies all four column tiles: 48 instructions of 32 cycles.  So a row of H is loaded and split once per 128 rows, a
// coefficient once per 128 feature columns.  A piece's sums go to the workspace; a second kernel adds the pieces of a block in
// order.
//
// Bound: the matrix cores beside 230 vector instructions a step; a loop of these matrix instructions alone reaches 2.05 PFLOP/s
// here on random operands, the library's 8192^3 bf16 product 1.1-1.4.  Measured (30 000 rows of 98 000 columns, 608 columns of H, 564
// rows of 6 144 entries and more, 1.0 TFLOP in the six products): fp32 panels 0.81 ms; here with loads one step ahead, non-temporal
// coefficients and an interval's chunks of one block next to each other 0.54; its blocks of one chunk next to each other and
// coefficients left in the L2 0.48; loads two steps ahead, for which the columns come from LDS (a load waited for is one all older
// ones are waited for with) 0.42 = 1.08 PFLOP/s.  One workgroup per CU instead of two 0.47-0.53; splitting between the
// matrix instructions instead of after them: no change.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <new>
#include <type_traits>
#include <vector>

#include "adaqp.h"
#include "common.hpp"

namespace adaqp {
namespace {

constexpr int kBlockRows = ADAQP_SPMM_BLOCK_ROWS;
constexpr int kStepCols = ADAQP_SPMM_BLOCK_STEP;    // columns of a step: two matrix instructions deep
constexpr int kRowGroups = kBlockRows / 32;         // one per wave
constexpr int kMostSteps = 128;                     // of a piece
constexpr int kTiles = 4;                           // column tiles of 32 of a workgroup, one per wave to load
constexpr int kChunk = kTiles * 32;                 // feature columns of a workgroup
constexpr int kStrip = kWave * 4;                   // feature columns of a workgroup of the sums
constexpr int kXcds = 8;
constexpr int kRawBuffer = 0x00020000;              // buffer resource, last word: raw 32-bit data, no swizzle
constexpr int64_t kMostBytes = 0xFFFF0000;          // of H: offsets are kept in 32 bits
constexpr int64_t kMostCols = 1 << 24, kMostPitch = 1 << 22;    // and are products of 24-bit factors (columns, bytes of a pitch)

static_assert(kRowGroups == kWavesPerBlock && kTiles == kWavesPerBlock && kStepCols == 32, "one wave per row group and tile");

typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef int int4_t __attribute__((ext_vector_type(4)));
typedef uint32_t uint32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

struct BlockArgs {
    const int32_t *rows;        // [n_blocks * 128], -1: none
    const int32_t *step_ptr;    // [n_blocks * n_pieces + 1]
    const int32_t *cols;        // [n_steps][32]
    const float *table;         // [n_steps][4 row groups][2][64 lanes][8]
    int32_t n_blocks, n_pieces, n_steps;
    const float *H;
    int32_t n_cols;
    int64_t ldh;
    int32_t dim, wdim;          // wdim = dim rounded up to whole 128-byte lines
    float *out;
    int64_t ldo;
    int64_t row_begin, row_end;
    float *partial;             // [n_blocks * n_pieces][128][wdim]
};

// Eight values of a lane as the three operands of a matrix instruction.
struct Operand {
    bf16x8_t hi, mid, lo;
};

// hi is the value rounded to bf16, mid the remainder rounded, lo what is left of that, 7 bits or fewer.  (A value that rounds to
// infinity, 3.39e38 and above, has a NaN for remainder: spmm_block_sum_kernel takes such sums again.)  Two values at a time; a
// subtraction is a dot product of a pair with (-1, 0) or (0, -1), which takes the bf16 as it is.
__device__ __forceinline__ Operand split8(const float (&x)[8])
{
    // from registers: as an inline constant the instruction takes -1.0 for the pair (0, -1), whichever of the two is meant
    uint32_t minus_first = 0x0000BF80u, minus_second = 0xBF800000u;
    asm("" : "+s"(minus_first), "+s"(minus_second));
    const bf16x2_t first = __builtin_bit_cast(bf16x2_t, minus_first), second = __builtin_bit_cast(bf16x2_t, minus_second);
    uint32x4_t hi, mid, lo;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x0 = x[2 * j], x1 = x[2 * j + 1];
        const bf16x2_t h = __builtin_convertvector((float2_t{x0, x1}), bf16x2_t);
        hi[j] = __builtin_bit_cast(uint32_t, h);
        const float r0 = __builtin_amdgcn_fdot2_f32_bf16(h, first, x0, false);
        const float r1 = __builtin_amdgcn_fdot2_f32_bf16(h, second, x1, false);
        const bf16x2_t m = __builtin_convertvector((float2_t{r0, r1}), bf16x2_t);
        mid[j] = __builtin_bit_cast(uint32_t, m);
        const float l0 = __builtin_amdgcn_fdot2_f32_bf16(m, first, r0, false);
        const float l1 = __builtin_amdgcn_fdot2_f32_bf16(m, second, r1, false);
        lo[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t{l0, l1}), bf16x2_t));
    }
    return Operand{__builtin_bit_cast(bf16x8_t, hi), __builtin_bit_cast(bf16x8_t, mid), __builtin_bit_cast(bf16x8_t, lo)};
}

// A step's rows of H as operands, for two steps, and the columns of all steps.
struct Stage {
    bf16x8_t part[2][2][kTiles][3][kWave];          // [buffer][half of the step][tile][hi, mid, lo][lane]
    int4_t cols[kMostSteps * kStepCols / 4];
};
static_assert(sizeof(Stage) <= 64 * 1024, "two workgroups fit a CU");

// LDS only: loads from memory stay in flight across the barrier.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One piece x T column tiles from feature column c_begin on.
//
// v_mfma_f32_32x32x16_bf16 computes D[32][32] += A[32][16] * B[16][32] with A's elements (m, 8h .. 8h + 7) in lane 32h + m,
// B's elements (8h .. 8h + 7, n) in lane 32h + n, and D's element (8 * (v / 4) + 4 * (lane / 32) + v % 4, lane % 32) in value
// v of the lane's 16.  Here m = row of the row group, n = feature column of the tile, k = column of half a step.
template <int T>
__device__ __forceinline__ void block_piece(const BlockArgs &a, Stage &stage, int32_t piece, int32_t s0, int32_t s1, int32_t c_begin)
{
    const int lane = threadIdx.x & (kWave - 1), half = lane >> 5, n = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int tile = min(wave, T - 1);              // the wave's to load; in a narrower chunk some take the last one again
    const int32_t last = s1 - 1;

    const auto rows_of_h = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.H), 0,
                                                             (int)(uint32_t)((int64_t)a.n_cols * a.ldh * 4), kRawBuffer);
    const uint32_t pitch = (uint32_t)a.ldh * 4u, last_col = (uint32_t)a.n_cols - 1u;
    const uint32_t lane_off = (uint32_t)(c_begin + tile * 32 + n) * 4u;

    // Loads are two steps ahead: two sets of registers in turn (P, for even and odd steps).
    float x[2][2][8];
    float4_t coef[2][2][2];
    auto request_rows = [&](auto P, int32_t s) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int4_t cols = stage.cols[(s - s0) * (kStepCols / 4) + k * 4 + half * 2 + q];
#pragma unroll
                for (int j = 0; j < 4; ++j) {       // a corrupt plan cannot lead outside H
                    const uint32_t c = min((uint32_t)cols[j], last_col);
                    x[P][k][q * 4 + j] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(rows_of_h, (int)(__umul24(c, pitch) + lane_off), 0, 0));
                }
            }
    };
    auto put_rows = [&](auto P) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const Operand o = split8(x[P][k]);
            stage.part[P][k][wave][0][lane] = o.hi;
            stage.part[P][k][wave][1][lane] = o.mid;
            stage.part[P][k][wave][2][lane] = o.lo;
        }
    };
    auto request_coef = [&](auto P, int32_t s, int k) {
        const float *from = a.table + ((((int64_t)s * kRowGroups + wave) * 2 + k) * kWave + lane) * 8;
#pragma unroll
        for (int q = 0; q < 2; ++q) coef[P][k][q] = *(reinterpret_cast<const float4_t *>(from) + q);
    };

    float16_t high[T], low[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) high[t][v] = low[t][v] = 0.0f;

    // Nothing in a step is behind a condition, steps past the last are the last one again: the compiler counts the loads in
    // flight over all paths, and waits for the youngest where one path has fewer.
    constexpr std::integral_constant<int, 0> even;
    constexpr std::integral_constant<int, 1> odd;
    for (int32_t i = threadIdx.x; i < (s1 - s0) * (kStepCols / 4); i += kBlock)
        stage.cols[i] = reinterpret_cast<const int4_t *>(a.cols)[(int64_t)s0 * (kStepCols / 4) + i];
    lds_barrier();
    request_rows(even, s0);
#pragma unroll
    for (int k = 0; k < 2; ++k) request_coef(even, s0, k);
    request_rows(odd, min(s0 + 1, last));
#pragma unroll
    for (int k = 0; k < 2; ++k) request_coef(odd, min(s0 + 1, last), k);
    put_rows(even);
    request_rows(even, min(s0 + 2, last));
    auto step = [&](auto P, auto other, int32_t s) {        // P: parity of s - s0
        lds_barrier();                              // the step's rows are there, and nobody reads the other buffer any more
        bf16x8_t b[2][3];                           // of a tile, and of the next one: read before the matrix instructions
        auto fetch = [&](int i) {
#pragma unroll
            for (int q = 0; q < 3; ++q) b[i & 1][q] = stage.part[P][i / T][i % T][q][lane];
        };
        fetch(0);
        Operand A;
#pragma unroll
        for (int i = 0; i < 2 * T; ++i) {
            if (i % T == 0) {
                const int k = i / T;
                float c8[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) c8[j] = coef[P][k][j / 4][j % 4];
                A = split8(c8);
                request_coef(P, min(s + 2, last), k);
            }
            if (i + 1 < 2 * T) fetch(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8_t hi = b[i & 1][0], mid = b[i & 1][1], lo = b[i & 1][2];
            float16_t &up = high[i % T], &down = low[i % T];
            down = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.lo, hi, down, 0, 0, 0);
            up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.hi, hi, up, 0, 0, 0);
            down = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.hi, lo, down, 0, 0, 0);
            down = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.mid, mid, down, 0, 0, 0);
            down = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.mid, hi, down, 0, 0, 0);
            down = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.hi, mid, down, 0, 0, 0);
        }
        put_rows(other);
        request_rows(other, min(s + 3, last));
    };
    for (int32_t s = s0; s < s1; s += 2) {
        step(even, odd, s);
        if (s + 1 < s1) step(odd, even, s + 1);
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = wave * 32 + 8 * (v / 4) + 4 * half + v % 4;
            __builtin_nontemporal_store(high[t][v] + low[t][v],
                                        a.partial + ((int64_t)piece * kBlockRows + m) * a.wdim + c_begin + t * 32 + n);
        }
}

// Workgroup i runs on XCD i mod 8, which takes every eighth interval of the columns: all blocks of a chunk of feature columns, which
// share the rows of H, then the next chunk of the interval, which shares the coefficients.
__global__ __launch_bounds__(kBlock, 2) void spmm_block_kernel(const BlockArgs a, int32_t n_chunks)
{
    __shared__ Stage stage;
    const uint32_t xcd = blockIdx.x % kXcds, task = blockIdx.x / kXcds;
    const uint32_t per_interval = (uint32_t)a.n_blocks * (uint32_t)n_chunks;
    const uint32_t interval = task / per_interval * kXcds + xcd;
    if (interval >= (uint32_t)a.n_pieces) return;
    const uint32_t chunk = task % per_interval / (uint32_t)a.n_blocks, block = task % (uint32_t)a.n_blocks;
    const int32_t piece = (int32_t)(block * (uint32_t)a.n_pieces + interval);
    const int32_t s0 = max(0, min(a.step_ptr[piece], a.n_steps)), s1 = max(s0, min(min(a.step_ptr[piece + 1], a.n_steps), s0 + kMostSteps));
    if (s0 == s1) return;                           // the whole workgroup; the sums skip the piece too
    const int32_t c_begin = (int32_t)chunk * kChunk, left = (a.wdim - c_begin) / 32;
    if (left >= 4) block_piece<4>(a, stage, piece, s0, s1, c_begin);
    else if (left == 3) block_piece<3>(a, stage, piece, s0, s1, c_begin);
    else if (left == 2) block_piece<2>(a, stage, piece, s0, s1, c_begin);
    else block_piece<1>(a, stage, piece, s0, s1, c_begin);
}

// One wave's share of a row's sum in plain fp32, from the pieces wave, wave + 4, ...: only the columns that the row lists, all of
// whose places in the table hold something other than +0 (0 x inf is NaN where an entry has the coefficient 0, too).
__device__ float4_t listed_columns(const BlockArgs &a, int32_t first, int32_t m, int32_t wave, int32_t lane, int32_t c, bool live)
{
    float4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int32_t p = wave; p < a.n_pieces; p += kWavesPerBlock) {
        const int32_t s0 = max(0, min(a.step_ptr[first + p], a.n_steps)), s1 = max(s0, min(min(a.step_ptr[first + p + 1], a.n_steps), s0 + kMostSteps));
        for (int32_t s = s0; s < s1; ++s) {
            const int32_t k = lane % kStepCols;                     // lane k: the step's column k
            const float alpha = a.table[((((int64_t)s * kRowGroups + m / 32) * 2 + k / 16) * kWave + (k / 8 % 2) * 32 + m % 32) * 8 + k % 8];
            const int32_t col = (int32_t)min((uint32_t)a.cols[(int64_t)s * kStepCols + k], (uint32_t)a.n_cols - 1u);
            for (uint32_t lists = (uint32_t)__ballot(__builtin_bit_cast(uint32_t, alpha) != 0); lists; lists &= lists - 1) {
                const int32_t q = __builtin_ctz(lists);
                const float w = __shfl(alpha, q);
                const int64_t from = __shfl(col, q);
                if (live) {
                    const float4_t x = *reinterpret_cast<const float4_t *>(a.H + from * a.ldh + c);
#pragma unroll
                    for (int t = 0; t < 4; ++t) sum[t] += w * x[t];
                }
            }
        }
    }
    return sum;
}

// out[row of a block] = sum of the block's pieces, in a fixed order; whole lines, row padding zero.  A workgroup per row and
// strip of 256 columns; its four waves take every fourth piece each and their sums are added in wave order.
//
// An infinity or NaN in H makes every row of the piece NaN there (0 x inf, and inf has no remainder to split off), so sums that
// are not finite are taken again from the columns that the row itself lists: rows without such a column keep their sums, the
// others get what fp32 gives.
__global__ __launch_bounds__(kBlock) void spmm_block_sum_kernel(const BlockArgs a, int32_t n_strips)
{
    __shared__ float4_t part[2][kWavesPerBlock][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t r = blockIdx.x / (uint32_t)n_strips;              // block * 128 + m
    const int32_t strip = (int32_t)(blockIdx.x % (uint32_t)n_strips);
    const int64_t row = a.rows[r];
    if (row < a.row_begin || row >= a.row_end) return;              // the whole workgroup: no barrier is skipped by a part
    const int32_t first = (int32_t)(r / kBlockRows) * a.n_pieces, m = (int32_t)(r % kBlockRows);
    const int32_t c = strip * kStrip + lane * 4;
    const bool live = c < a.wdim;
    constexpr int kAhead = 8;
    float4_t sum = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int32_t p = wave; p < a.n_pieces; p += kAhead * kWavesPerBlock) {
        float4_t x[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int32_t pq = p + q * kWavesPerBlock;
            x[q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if (live && pq < a.n_pieces && a.step_ptr[first + pq] < a.step_ptr[first + pq + 1])
                x[q] = __builtin_nontemporal_load(
                    reinterpret_cast<const float4_t *>(a.partial + ((int64_t)(first + pq) * kBlockRows + m) * a.wdim + c));
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) sum += x[q];
    }
    auto add_waves = [&](const float4_t (&of)[kWavesPerBlock][kWave]) {
        float4_t total = of[0][lane];
#pragma unroll
        for (int w = 1; w < kWavesPerBlock; ++w) total += of[w][lane];
        return total;
    };
    part[0][wave][lane] = sum;
    __syncthreads();
    float4_t total = add_waves(part[0]);                            // in every wave: all of them take the branch below, or none
    bool again[4], any = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (c + k >= a.dim) total[k] = 0.0f;                        // row padding
        again[k] = !(__builtin_fabsf(total[k]) < __builtin_inff());
        any |= again[k];
    }
    if (__ballot(any) != 0) {
        part[1][wave][lane] = listed_columns(a, first, m, wave, lane, c, live);
        __syncthreads();
        const float4_t exact = add_waves(part[1]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (again[k]) total[k] = exact[k];
    }
    if (wave == 0 && live) __builtin_nontemporal_store(total, reinterpret_cast<float4_t *>(a.out + row * a.ldo + c));
}

// The table: zeros, then the coefficient of every entry of the blocks' rows at its column's place, -0 for a coefficient of 0: a
// product of it adds nothing, as the plain zeros do, and the column stays one that the row lists.
__global__ __launch_bounds__(kBlock) void block_table_clear_kernel(float4_t *table, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        table[i] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
}

// A workgroup per row of a block.  copied: NULL, or what val held for the range's entries when the table was written last: entries that are
// still the same are left alone, the others are written to both.  21.8 M entries of 1 555 rows: 0.085 ms where nothing has changed (the two
// reads, 2.1 TB/s, a chain of them per row), 1.1 where all has (a search over the piece's columns and a scattered write each).
__global__ __launch_bounds__(kBlock) void block_table_fill_kernel(const BlockArgs a, float *table, int32_t col_begin, int32_t width,
                                                                  const int64_t *rowptr, const int32_t *col, const float *val, int64_t nnz,
                                                                  float *copied)
{
    const int64_t row = a.rows[blockIdx.x];
    if (row < a.row_begin || row >= a.row_end) return;
    const int32_t block = (int32_t)(blockIdx.x / kBlockRows), m = (int32_t)(blockIdx.x % kBlockRows);
    const int64_t base = max((int64_t)0, min(rowptr[a.row_begin], nnz));
    const int64_t lo = max(base, min(rowptr[row], nnz)), hi = max(lo, min(rowptr[row + 1], nnz));
    auto place = [&](int64_t j, float coefficient) {
        const int32_t c = col[j];
        if (c < col_begin) return;
        const int32_t interval = (c - col_begin) / width;
        if (interval >= a.n_pieces) return;
        const int32_t piece = block * a.n_pieces + interval;
        const int32_t s0 = max(0, min(a.step_ptr[piece], a.n_steps)), s1 = max(s0, min(a.step_ptr[piece + 1], a.n_steps));
        // the first of the piece's columns that is not below c (behind the last one it is repeated)
        int64_t from = (int64_t)s0 * kStepCols, to = (int64_t)s1 * kStepCols;
        const int64_t end = to;
        while (from < to) {
            const int64_t mid = (from + to) / 2;
            if (a.cols[mid] < c) from = mid + 1;
            else to = mid;
        }
        if (from >= end || a.cols[from] != c) return;               // not of this plan
        const int64_t s = from / kStepCols;
        const int32_t k = (int32_t)(from % kStepCols), lane = (k / 8 % 2) * 32 + m % 32;
        table[((((s * kRowGroups + m / 32) * 2 + k / 16) * kWave) + lane) * 8 + k % 8] = coefficient == 0.0f ? -0.0f : coefficient;
    };
    constexpr int kAhead = 4;                                       // loads of a lane in flight together
    for (int64_t j = lo + threadIdx.x; j < hi; j += kAhead * kBlock) {
        uint32_t now[kAhead], was[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t at = min(j + q * kBlock, hi - 1);
            now[q] = __builtin_bit_cast(uint32_t, val[at]);
            was[q] = copied ? __builtin_bit_cast(uint32_t, copied[at - base]) : ~now[q];
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t at = j + q * kBlock;
            if (at >= hi || now[q] == was[q]) continue;
            const float coefficient = __builtin_bit_cast(float, now[q]);
            if (copied) copied[at - base] = coefficient;
            place(at, coefficient);
        }
    }
}

int64_t blocks_bytes(int64_t n_blocks, int64_t n_pieces, int32_t dim)
{
    const int64_t wdim = ((int64_t)dim + 31) / 32 * 32;
    return (n_blocks * n_pieces * kBlockRows * wdim * 4 + 255) / 256 * 256;
}

// Of the two launches; a launch has fewer than 2^31 threads.
constexpr int64_t kMostWorkgroups = 0x7FFFFFFF / kBlock;

int64_t product_workgroups(const adaqp_spmm_blocks *p, int32_t dim)
{
    return ((int64_t)p->n_pieces + kXcds - 1) / kXcds * kXcds * p->n_blocks * (((int64_t)dim + kChunk - 1) / kChunk);
}

int64_t sum_workgroups(int64_t n_blocks, int64_t dim) { return n_blocks * kBlockRows * ((dim + kStrip - 1) / kStrip); }

// Intervals of the columns.  A round is what the GPU's 512 resident workgroups take at a time; an interval costs each of its
// workgroups about four steps to start and end, and its sums a tenth of a step's time per block to write and read.
int32_t choose_pieces(int64_t n_blocks, int64_t n_chunks, int64_t n_cols)
{
    const int64_t steps = (n_cols + kStepCols - 1) / kStepCols;
    int32_t best = 0;
    double best_cost = 0.0;
    const int64_t fewest = (steps / kMostSteps + kXcds) / kXcds * kXcds;          // pieces of kMostSteps at most
    for (int64_t p = fewest; p <= fewest + 256; p += kXcds) {
        const int64_t rounds = (p / kXcds * n_blocks * n_chunks + 63) / 64;
        const double cost = (double)rounds * (double)((steps + p - 1) / p + 4) + 0.1 * (double)p * (double)n_blocks;
        if (p == fewest || cost < best_cost) {
            best = (int32_t)p;
            best_cost = cost;
        }
    }
    return best;
}

int check_blocks(const adaqp_spmm_blocks *p)
{
    if (p->n_blocks < 0 || p->n_pieces < 0 || p->n_steps < 0) return ADAQP_EINVAL;
    if (p->n_blocks == 0) return ADAQP_OK;
    if (p->n_pieces == 0 || p->n_pieces > (1 << 16) || p->n_steps > INT32_MAX - 1 || p->col_begin < 0 || p->piece_width < 1) return ADAQP_EINVAL;
    if (p->n_blocks > INT32_MAX / kBlockRows || (int64_t)p->n_blocks * p->n_pieces > INT32_MAX - 1) return ADAQP_ESIZE;
    if (!p->rows_dev || !p->step_ptr_dev || !p->cols_dev || !p->table_dev) return ADAQP_EINVAL;
    if (!aligned_to(p->rows_dev, 4) || !aligned_to(p->step_ptr_dev, 4) || !aligned_to(p->cols_dev, 16) || !aligned_to(p->table_dev, 16))
        return ADAQP_EINVAL;
    return ADAQP_OK;
}

BlockArgs block_args(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end)
{
    BlockArgs a = {};
    a.rows = p->rows_dev;
    a.step_ptr = p->step_ptr_dev;
    a.cols = p->cols_dev;
    a.table = p->table_dev;
    a.n_blocks = p->n_blocks;
    a.n_pieces = p->n_pieces;
    a.n_steps = (int32_t)p->n_steps;
    a.row_begin = row_begin;
    a.row_end = row_end;
    return a;
}

}  // namespace
}  // namespace adaqp

using namespace adaqp;

extern "C" int adaqp_plan_spmm_blocks(const int64_t *rowptr_host, const int32_t *col_host, int64_t row_begin, int64_t row_end,
                                      int64_t n_cols, int32_t dim, int32_t min_row_len, int64_t *sizes_inout,
                                      int32_t *tile_off_inout, int32_t *rows_out, int32_t *step_ptr_out, int32_t *cols_out)
try {
    if (row_begin < 0 || row_end < row_begin || n_cols < 0 || n_cols > INT32_MAX || dim <= 0 || min_row_len < 1) return ADAQP_EINVAL;
    if (!rowptr_host || !sizes_inout) return ADAQP_EINVAL;
    const bool fill = rows_out != nullptr;
    if (fill && (!step_ptr_out || !cols_out)) return ADAQP_EINVAL;

    std::vector<int64_t> heavy;                     // longest first
    for (int64_t r = row_begin; r < row_end; ++r) {
        const int64_t s = rowptr_host[r], e = rowptr_host[r + 1];
        if (s < 0 || e < s || e - s > INT32_MAX) return ADAQP_EINVAL;
        if (e - s >= min_row_len) heavy.push_back(r);
    }
    if (!heavy.empty() && !col_host) return ADAQP_EINVAL;
    std::stable_sort(heavy.begin(), heavy.end(), [&](int64_t x, int64_t y) {
        return rowptr_host[x + 1] - rowptr_host[x] > rowptr_host[y + 1] - rowptr_host[y];
    });
    const int64_t n_heavy = (int64_t)heavy.size(), n_blocks = (n_heavy + kBlockRows - 1) / kBlockRows;
    if (n_blocks > INT32_MAX / kBlockRows) return ADAQP_ESIZE;
    int32_t lo = INT32_MAX, hi = -1;
    for (const int64_t r : heavy) {
        int32_t before = -1;                        // columns are ascending and distinct
        for (int64_t j = rowptr_host[r]; j < rowptr_host[r + 1]; ++j) {
            const int32_t c = col_host[j];
            if (c <= before || c >= n_cols) return ADAQP_EINVAL;
            before = c;
        }
        if (before < 0) continue;
        lo = std::min(lo, col_host[rowptr_host[r]]);
        hi = std::max(hi, before);
    }
    if (hi < 0) lo = 0;
    const int64_t span = std::max<int64_t>((int64_t)hi + 1 - lo, 1);
    const int64_t n_chunks = ((int64_t)dim + kChunk - 1) / kChunk;
    const int32_t n_pieces = n_blocks ? choose_pieces(n_blocks, n_chunks, span) : 0;
    const int32_t width = n_blocks ? (int32_t)((span + n_pieces - 1) / n_pieces) : 1;
    if (n_blocks * n_pieces > INT32_MAX - 1) return ADAQP_ESIZE;
    if (fill && (sizes_inout[0] != n_heavy || sizes_inout[1] != n_blocks || sizes_inout[2] != n_pieces || sizes_inout[4] != lo ||
                 sizes_inout[5] != width))
        return ADAQP_EINVAL;                        // the arrays were sized for another plan

    std::vector<uint8_t> used((size_t)n_cols, 0);
    int64_t n_steps = 0;
    for (int64_t b = 0; b < n_blocks; ++b) {
        const int64_t m_end = std::min<int64_t>(kBlockRows, n_heavy - b * kBlockRows);
        for (int64_t m = 0; m < m_end; ++m) {
            const int64_t r = heavy[(size_t)(b * kBlockRows + m)];
            for (int64_t j = rowptr_host[r]; j < rowptr_host[r + 1]; ++j) used[(size_t)col_host[j]] = 1;
        }
        for (int32_t p = 0; p < n_pieces; ++p) {
            if (fill) step_ptr_out[b * n_pieces + p] = (int32_t)n_steps;
            const int64_t c0 = (int64_t)lo + (int64_t)p * width, c1 = std::min<int64_t>(c0 + width, (int64_t)hi + 1);
            int64_t at = 0;
            int32_t last = 0;
            for (int64_t c = c0; c < c1; ++c)
                if (used[(size_t)c]) {
                    used[(size_t)c] = 0;
                    last = (int32_t)c;
                    if (fill) {
                        if ((n_steps + at / kStepCols + 1) > sizes_inout[3]) return ADAQP_EINVAL;
                        cols_out[n_steps * kStepCols + at] = last;
                    }
                    ++at;
                }
            const int64_t steps = (at + kStepCols - 1) / kStepCols;
            if (fill)
                for (; at < steps * kStepCols; ++at) cols_out[n_steps * kStepCols + at] = last;
            n_steps += steps;
            if (n_steps > INT32_MAX / kStepCols) return ADAQP_ESIZE;
        }
    }
    if (!fill) {
        sizes_inout[0] = n_heavy;
        sizes_inout[1] = n_blocks;
        sizes_inout[2] = n_pieces;
        sizes_inout[3] = n_steps;
        sizes_inout[4] = lo;
        sizes_inout[5] = width;
        return ADAQP_OK;
    }
    if (n_steps != sizes_inout[3]) return ADAQP_EINVAL;
    step_ptr_out[n_blocks * n_pieces] = (int32_t)n_steps;
    for (int64_t k = 0; k < n_blocks * kBlockRows; ++k) rows_out[k] = k < n_heavy ? (int32_t)heavy[(size_t)k] : -1;
    if (tile_off_inout)
        for (const int64_t r : heavy)
            std::fill_n(tile_off_inout + (r - row_begin) * (ADAQP_SPMM_TILES + 1), ADAQP_SPMM_TILES + 1, -1);
    return ADAQP_OK;
} catch (const std::bad_alloc &) {           // nothing may be thrown through a C entry
    return ADAQP_ESIZE;
}

// A row of a block costs every column of the block: at 1.08 PFLOP/s and 7.5 ps per entry and line in tile order 4.5 % of the columns break
// even, where there are many lines.  Which rows can be worth it; whether they are, adaqp_spmm_blocks_save says.
constexpr int64_t kColumnsPerEntry = 20, kFewestRows = 256;

extern "C" int32_t adaqp_spmm_blocks_min_row(int64_t n_cols)
{
    return (int32_t)std::min<int64_t>(std::max<int64_t>(n_cols / kColumnsPerEntry, 64), INT32_MAX);
}

extern "C" int32_t adaqp_spmm_blocks_pay(int64_t n_rows_taken, int64_t n_cols, int64_t ldh)
{
    return n_rows_taken >= kFewestRows && n_cols > 0 && n_cols <= kMostCols && ldh < kMostPitch && n_cols * ldh <= kMostBytes / 4 &&
           sum_workgroups((n_rows_taken + kBlockRows - 1) / kBlockRows, ldh) <= kMostWorkgroups ? 1 : 0;
}

// What the entries cost in tile order against what their blocks cost: a step is a load and a split of coefficients per chunk of feature
// columns and of the rows of H per line beside its matrix instructions, and less of it shows where another range's entries are walked at
// the same time.
// One after the other: 228 launches of 24 000 and 90 000 columns, 130 to 1 792 rows that list 5.5, 12 or 25 % of them, 32 to 602 columns of H,
// beside 10 000 rows of 100 entries.  Geometric mean against no blocks 1.16, the largest loss 10 % (blocks for every 256 rows: 1.04, 2.05 times
// as slow at worst).  384 rows of 12 %, 90 000 columns, 64 columns of H 87 -> 112 us (no), 96 141 -> 129 (yes), 602 702 -> 520 (yes);
// 256 rows of 12 %, 24 000 columns, 128 columns of H 65 -> 67 (no), 256 109 -> 95 (yes).
// Beside: 133 forward steps of 6 000 to 58 000 rows, 130 to 450 entries per row, Zipf and log-normal, 32 to 602 columns of H.  Geometric mean
// against no blocks 1.258, the largest loss 8 % (the better of both each time 1.264, blocks for every 256 rows 1.213 and 54 %).
// 20 000 rows, 9 M entries, log-normal, 64 columns 154 -> 171 us (no); 10 000 rows, 4.5 M entries, log-normal, 400 columns 400 -> 324 (yes),
// 32 70 -> 108 (no).
extern "C" int32_t adaqp_spmm_blocks_save(int64_t n_entries, int64_t n_steps, int32_t dim, int32_t beside)
{
    if (n_entries <= 0 || n_steps <= 0 || dim <= 0) return 0;
    const double lines = (double)(((int64_t)dim + 31) / 32), chunks = (double)(((int64_t)dim + kChunk - 1) / kChunk);
    const double entries_ns = 5.6e-3 * lines * (double)n_entries, step_ns = beside ? 2.0 * chunks + 0.35 * lines : 2.7 * chunks + 0.75 * lines;
    return entries_ns > 15e3 + step_ns * (double)n_steps ? 1 : 0;
}

// A table takes 16 KB per step, however few of its places are filled: ten times what the entries of rows at the threshold take.  Four times
// the col and val of the range leaves 58 000 rows with 28 M entries what they have (2.0 and 2.4 times); 64 MB are never too many.
extern "C" int64_t adaqp_spmm_blocks_most_steps(int64_t nnz)
{
    constexpr int64_t kStepBytes = (int64_t)kStepCols * kBlockRows * 4;
    return std::max<int64_t>((nnz < 0 ? 0 : nnz) / (kStepBytes / (4 * 8)), ((int64_t)64 << 20) / kStepBytes);
}

extern "C" int64_t adaqp_spmm_blocks_table_floats(int64_t n_steps) { return n_steps < 0 ? -1 : n_steps * kStepCols * kBlockRows; }

namespace {

// copied: of adaqp_update_spmm_blocks, NULL to write the whole table.
int write_table(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const int64_t *rowptr_dev, const int32_t *col_dev,
                const float *val_dev, int64_t nnz, float *copied_dev, hipStream_t st)
{
    if (!p) return ADAQP_EINVAL;
    const int rc = check_blocks(p);
    if (rc != ADAQP_OK) return rc;
    if (row_begin < 0 || row_end < row_begin || nnz < 0) return ADAQP_EINVAL;
    if (p->n_blocks == 0 || p->n_steps == 0) return ADAQP_OK;
    if (!rowptr_dev || !aligned_to(rowptr_dev, 8) || (nnz > 0 && (!col_dev || !val_dev || !aligned_to(col_dev, 4) || !aligned_to(val_dev, 4))))
        return ADAQP_EINVAL;
    const BlockArgs a = block_args(p, row_begin, row_end);
    if (!copied_dev) {
        const int64_t vectors = adaqp_spmm_blocks_table_floats(p->n_steps) / 4;
        hipLaunchKernelGGL(block_table_clear_kernel, dim3((unsigned)std::min<int64_t>((vectors + kBlock - 1) / kBlock, 16384)), dim3(kBlock), 0, st,
                           reinterpret_cast<float4_t *>(p->table_dev), vectors);
        ADAQP_HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(block_table_fill_kernel, dim3((unsigned)(p->n_blocks * kBlockRows)), dim3(kBlock), 0, st, a, p->table_dev,
                       p->col_begin, p->piece_width, rowptr_dev, col_dev, val_dev, nnz, copied_dev);
    ADAQP_HIP_TRY(hipGetLastError());
    return ADAQP_OK;
}

}  // namespace

extern "C" int adaqp_fill_spmm_blocks(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const int64_t *rowptr_dev,
                                      const int32_t *col_dev, const float *val_dev, int64_t nnz, void *stream)
{
    return write_table(p, row_begin, row_end, rowptr_dev, col_dev, val_dev, nnz, nullptr, (hipStream_t)stream);
}

extern "C" int adaqp_update_spmm_blocks(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const int64_t *rowptr_dev,
                                        const int32_t *col_dev, const float *val_dev, int64_t nnz, float *copied_dev, void *stream)
{
    if (!copied_dev || !aligned_to(copied_dev, 4)) return ADAQP_EINVAL;
    return write_table(p, row_begin, row_end, rowptr_dev, col_dev, val_dev, nnz, copied_dev, (hipStream_t)stream);
}

extern "C" int adaqp_spmm_blocks_workspace_bytes(int32_t n_blocks, int32_t n_pieces, int32_t dim, int64_t *bytes_out)
{
    if (!bytes_out || n_blocks < 0 || n_pieces < 0 || dim <= 0) return ADAQP_EINVAL;
    if ((int64_t)n_blocks * n_pieces > INT32_MAX - 1) return ADAQP_ESIZE;
    *bytes_out = blocks_bytes(n_blocks, n_pieces, dim);
    return ADAQP_OK;
}

int adaqp::check_blocks_call(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const float *H_dev, int64_t n_cols, int64_t ldh,
                             int32_t dim, const float *out_dev, int64_t ldo)
{
    if (!p) return ADAQP_EINVAL;
    const int rc = check_blocks(p);
    if (rc != ADAQP_OK) return rc;
    if (row_begin < 0 || row_end < row_begin || dim <= 0 || ldh < dim || ldo < dim || n_cols < 0) return ADAQP_EINVAL;
    if (p->n_blocks == 0 || row_end == row_begin) return ADAQP_OK;
    if (!H_dev || !out_dev || n_cols == 0) return ADAQP_EINVAL;
    if (n_cols > kMostCols || ldh >= kMostPitch || n_cols * ldh > kMostBytes / 4) return ADAQP_ESIZE;
    if (ldh % 32 != 0 || ldo % 32 != 0 || !aligned_to(H_dev, 128) || !aligned_to(out_dev, 128)) return ADAQP_EINVAL;
    if (product_workgroups(p, dim) > kMostWorkgroups || sum_workgroups(p->n_blocks, dim) > kMostWorkgroups) return ADAQP_ESIZE;
    return ADAQP_OK;
}

extern "C" int adaqp_spmm_csr_blocks(const adaqp_spmm_blocks *p, int64_t row_begin, int64_t row_end, const float *H_dev,
                                     int64_t n_cols, int64_t ldh, int32_t dim, float *out_dev, int64_t ldo,
                                     void *workspace_dev, int64_t workspace_bytes, void *stream)
{
    const int rc = check_blocks_call(p, row_begin, row_end, H_dev, n_cols, ldh, dim, out_dev, ldo);
    if (rc != ADAQP_OK || p->n_blocks == 0 || row_end == row_begin) return rc;
    const int64_t need = blocks_bytes(p->n_blocks, p->n_pieces, dim);
    if (!workspace_dev || !aligned_to(workspace_dev, 256)) return ADAQP_EINVAL;
    if (workspace_bytes < need) return ADAQP_ESIZE;

    BlockArgs a = block_args(p, row_begin, row_end);
    a.H = H_dev;
    a.n_cols = (int32_t)n_cols;
    a.ldh = ldh;
    a.dim = dim;
    a.wdim = (dim + 31) / 32 * 32;
    a.out = out_dev;
    a.ldo = ldo;
    a.partial = reinterpret_cast<float *>(workspace_dev);
    const int64_t n_chunks = (a.wdim + kChunk - 1) / kChunk, n_strips = (a.wdim + kStrip - 1) / kStrip;
    const int64_t blocks = product_workgroups(p, dim), sums = sum_workgroups(p->n_blocks, dim);
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(spmm_block_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, a, (int32_t)n_chunks);
    ADAQP_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(spmm_block_sum_kernel, dim3((unsigned)sums), dim3(kBlock), 0, st, a, (int32_t)n_strips);
    ADAQP_HIP_TRY(hipGetLastError());
    return ADAQP_OK;
}
