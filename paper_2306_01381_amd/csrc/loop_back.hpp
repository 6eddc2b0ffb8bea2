// The loop-back copy of the layer step and the table of received rows: in a launch of their own (layer.hip), or in workgroups of the launches
// around them.
#pragma once

#include <algorithm>

#include "common.hpp"

namespace adaqp {

struct CopyArgs {
    const uint8_t *from;
    uint8_t *to;
    int64_t bytes, units;       // whole units of 16, 4 or 1 bytes, as the addresses allow
    int32_t unit;
};

inline CopyArgs copy_args(const void *from, void *to, int64_t bytes)
{
    CopyArgs c;
    c.from = static_cast<const uint8_t *>(from);
    c.to = static_cast<uint8_t *>(to);
    c.bytes = bytes;
    c.unit = aligned_to(from, 16) && aligned_to(to, 16) ? 16 : (aligned_to(from, 4) && aligned_to(to, 4) ? 4 : 1);
    c.units = bytes / c.unit;
    return c;
}

// A launch has fewer than 2^32 threads: what 2^18 workgroups per buffer do not copy at one unit each they copy in turns.
constexpr int64_t kBesideBlocks = (int64_t)1 << 18;

// Both buffers in one launch (the runtime's copies cost the host more than a launch each, and the second one waits for the first).
struct LoopBack {
    CopyArgs packed, params;
    uint32_t blocks_packed, blocks_params;

    uint32_t blocks() const { return blocks_packed + blocks_params; }
};

constexpr LoopBack kNoLoopBack = {};

inline LoopBack loop_back_of(const adaqp_layer_desc *d)
{
    LoopBack c = kNoLoopBack;
    c.packed = copy_args(d->packed_dev, d->recv_packed_dev, d->packed_bytes);
    c.params = copy_args(d->params_dev, d->recv_params_dev, d->n_send * 2 * (int64_t)sizeof(float));
    auto blocks = [](const CopyArgs &of) { return (uint32_t)std::min((of.units + of.bytes % of.unit + kBlock - 1) / kBlock, kBesideBlocks); };
    c.blocks_packed = blocks(c.packed);
    c.blocks_params = blocks(c.params);
    return c;
}

// Thread i copies unit i, or one byte of what the whole units leave over.
__device__ __forceinline__ void copy_one(const CopyArgs &c, int64_t i)
{
    if (i >= c.units) {
        const int64_t at = c.units * c.unit + (i - c.units);
        if (at < c.bytes) c.to[at] = c.from[at];
    } else if (c.unit == 16) {
        reinterpret_cast<uint4 *>(c.to)[i] = reinterpret_cast<const uint4 *>(c.from)[i];
    } else if (c.unit == 4) {
        reinterpret_cast<uint32_t *>(c.to)[i] = reinterpret_cast<const uint32_t *>(c.from)[i];
    } else {
        c.to[i] = c.from[i];
    }
}

// The share of one of the copying workgroups, `block` of them, of `threads` threads.
__device__ __forceinline__ void copy_blocks(const LoopBack &c, uint32_t block, int32_t threads)
{
    const bool first = block < c.blocks_packed;
    if (block >= c.blocks_packed + c.blocks_params) return;
    const CopyArgs &of = first ? c.packed : c.params;
    const int64_t mine = first ? block : block - c.blocks_packed, blocks = first ? c.blocks_packed : c.blocks_params;
    const int64_t n = of.units + (of.bytes - of.units * of.unit);
    for (int64_t i = mine * threads + threadIdx.x; i < n; i += blocks * threads) copy_one(of, i);
}

// Where each row of feat is found: the place and slot of those that lie packed in the receive buffer, for the kernels that walk planned
// pieces.  Widths and offsets are read when they are used, as the quantisation reads them: a step follows what was written to them.
struct PackedRowArgs {
    const int32_t *slot_of_row;
    const uint8_t *bits;
    const int64_t *row_offset;
    int64_t n_rows, n_slots, packed_bytes;
    int32_t dim;
    uint32_t blocks;                    // workgroups of a launch that fill the table
    adaqp_packed_row *row;
};

constexpr PackedRowArgs kNoPackedRows = {};

inline PackedRowArgs packed_rows_of(const adaqp_layer_desc *d)
{
    return {d->slot_of_row_dev, d->bits_dev, d->row_offset_dev, d->n_feat_rows, d->n_send, d->packed_bytes, d->dim,
            (uint32_t)std::min((d->n_feat_rows + kBlock - 1) / kBlock, kBesideBlocks), d->packed_row_dev};
}

__device__ __forceinline__ adaqp_packed_row packed_row_at(const PackedRowArgs &p, int64_t r)
{
    const int32_t slot = p.slot_of_row[r];
    if (slot < 0 || slot >= p.n_slots) return {0, 0};
    const int32_t b = p.bits[slot];
    const int64_t at = p.row_offset[slot], stride = 4 * (((int64_t)p.dim * b + 31) >> 5);
    if (!(b == 2 || b == 4 || b == 8) || at < 0 || (at & 3) != 0 || at > p.packed_bytes - stride) return {0, 0};
    return {(uint32_t)at | (b == 2 ? 1u : (b == 4 ? 2u : 3u)), (uint32_t)slot};
}

// The share of one of the workgroups (of kBlock threads) that fill the table.
__device__ __forceinline__ void fill_packed_rows(const PackedRowArgs &p, uint32_t block)
{
    for (int64_t r = (int64_t)block * kBlock + threadIdx.x; r < p.n_rows; r += (int64_t)p.blocks * kBlock) p.row[r] = packed_row_at(p, r);
}

// The calls of adaqp.h with such workgroups in their launch.  Fewer than 2^25 messages: the launch stays below 2^32 threads.
constexpr int64_t kBesideMessages = (int64_t)1 << 25;
int quantize_pack_beside(const float *feat_dev, int64_t n_feat_rows, int64_t ld, int32_t dim, const int32_t *send_idx_dev,
                         const uint8_t *bits_dev, const int64_t *row_offset_dev, int64_t n_send, uint64_t seed, uint8_t *packed_dev,
                         int64_t packed_bytes, float *params_dev, const float *alpha_sq_dev, float *beta_dev, PackedRowArgs table, void *stream);
int unpack_dequant_beside(const uint8_t *packed_dev, int64_t packed_bytes, const float *params_dev, const uint8_t *bits_dev,
                          const int64_t *row_offset_dev, const int32_t *halo_idx_dev, const int32_t *order_dev, int64_t n_recv, int32_t dim,
                          float *feat_dev, int64_t n_feat_rows, int64_t ld, LoopBack copies, void *stream);
int unpack_dequant_add_beside(const uint8_t *packed_dev, int64_t packed_bytes, const float *params_dev, const uint8_t *bits_dev,
                              const int64_t *row_offset_dev, const int32_t *dst_idx_dev, int64_t n_recv, const int32_t *seg_order_dev,
                              const int64_t *seg_ptr_dev, int64_t n_seg, int32_t dim, float *grad_dev, int64_t n_grad_rows, int64_t ld,
                              LoopBack copies, void *stream);

}  // namespace adaqp
