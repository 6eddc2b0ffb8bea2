// Host side of libadaqp: status strings, the buffer layout of Sec. 5 "Implementation" (messages grouped by
// bit-width, groups concatenated per peer) and the layer step that overlaps the message path with the
// aggregation of the rows that do not depend on it (Sec. 3.1, Sec. 3.4 Fig. 7).
#include <stdio.h>
#include <string.h>

#include <algorithm>

#include "loop_back.hpp"
#include "spmm_common.hpp"
#include "host_sort.hpp"

namespace adaqp {

static thread_local char g_hip_error[256] = "";

int note_hip_error(hipError_t err, const char *what)
{
    snprintf(g_hip_error, sizeof(g_hip_error), "%s: %s", what, hipGetErrorString(err));
    return ADAQP_EHIP;
}

}  // namespace adaqp

using namespace adaqp;

extern "C" const char *adaqp_strerror(int status)
{
    switch (status) {
        case ADAQP_OK: return "ok";
        case ADAQP_EINVAL: return "invalid argument";
        case ADAQP_EBITS: return "bit-width outside {2, 4, 8}";
        case ADAQP_ESIZE: return "buffer or workspace too small, or size beyond a documented limit";
        case ADAQP_EHIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

extern "C" const char *adaqp_last_hip_error(void) { return g_hip_error; }

extern "C" int adaqp_version(void) { return ADAQP_VERSION; }

extern "C" int64_t adaqp_row_stride(int32_t dim, int32_t bits)
{
    if (dim <= 0 || !valid_bits(bits)) return -1;
    return 4 * (((int64_t)dim * bits + 31) / 32);
}

namespace {

// Whether peers ascend within [0, n_peers) and widths are ones that there are: checked without a branch per slot; only where something is
// wrong a second look says what comes first.
int check_slots(int64_t n, const uint8_t *bits_host, const int32_t *peer_of_slot_host, int32_t n_peers)
{
    bool ok = n == 0 || (peer_of_slot_host[0] >= 0 && peer_of_slot_host[n - 1] < n_peers);
    for (int64_t i = 0; i < n; ++i) ok &= (bits_host[i] == 2) | (bits_host[i] == 4) | (bits_host[i] == 8);
    for (int64_t i = 1; i < n; ++i) ok &= peer_of_slot_host[i - 1] <= peer_of_slot_host[i];
    for (int64_t i = 0; !ok && i < n; ++i) {
        if (!valid_bits(bits_host[i])) return ADAQP_EBITS;
        const int32_t p = peer_of_slot_host[i];
        if (p < 0 || p >= n_peers) return ADAQP_EINVAL;
        if (i > 0 && p < peer_of_slot_host[i - 1]) return ADAQP_EINVAL;
    }
    return ADAQP_OK;
}

// Places checked slots: width 2 first, then 4, then 8 inside a peer, input order kept.  place(i, k, byte): slot i comes to place k, its row to
// that byte.  The next place of a width waits for the slot before it (a store and a load of one address), so a peer's slots are walked in
// four parts at once, whose counts say where each begins (100 000 slots 192 -> 128 us); the few slots of a small peer in one.
constexpr int kWidths = 3;                                  // 2, 4, 8 >> 2

template <int PARTS, typename Place>
void place_peer(int64_t begin, int64_t end, const uint8_t *bits_host, const int64_t (&stride)[kWidths], int64_t *bytes, Place &place)
{
    const int64_t part = (end - begin) / PARTS;
    auto part_begin = [&](int q) { return q < PARTS ? begin + q * part : end; };
    int64_t next[PARTS][kWidths], byte_of_0[kWidths];       // byte_of_0 + k * stride: of place k
    for (int q = 0; q < PARTS; ++q) {
        int64_t n4 = 0, n8 = 0;
        for (int64_t i = part_begin(q); i < part_begin(q + 1); ++i) {
            n4 += bits_host[i] == 4;
            n8 += bits_host[i] == 8;
        }
        next[q][0] = part_begin(q + 1) - part_begin(q) - n4 - n8;
        next[q][1] = n4;
        next[q][2] = n8;
    }
    int64_t at = begin;
    for (int w = 0; w < kWidths; ++w) {
        byte_of_0[w] = *bytes - at * stride[w];
        for (int q = 0; q < PARTS; ++q) {
            const int64_t count = next[q][w];
            next[q][w] = at;
            at += count;
            *bytes += count * stride[w];
        }
    }
    auto place_one = [&](int q, int64_t i) {
        const int w = bits_host[i] >> 2;
        const int64_t k = next[q][w]++;
        place(i, k, byte_of_0[w] + k * stride[w]);
    };
    for (int64_t t = 0; t < part; ++t)
        for (int q = 0; q < PARTS; ++q) place_one(q, begin + q * part + t);
    for (int64_t i = begin + PARTS * part; i < end; ++i) place_one(PARTS - 1, i);
}

// Where a peer's slots end is looked for near where they begin: peers may be as many as slots (100 000 slots of as many peers, a search in all that
// follow and four parts for each 7.0 ms, so 1.35; 1 000 slots 3.2 and 0.17).
template <typename Place>
void place_slots(int64_t n, int32_t dim, const uint8_t *bits_host, const int32_t *peer_of_slot_host, int32_t n_peers, int64_t *peer_byte_ptr_out,
                 Place place)
{
    constexpr int64_t kSmall = 64;
    const int64_t stride[kWidths] = {adaqp_row_stride(dim, 2), adaqp_row_stride(dim, 4), adaqp_row_stride(dim, 8)};
    int64_t begin = 0, bytes = 0;
    for (int32_t p = 0; p < n_peers; ++p) {
        peer_byte_ptr_out[p] = bytes;
        int64_t end = begin;
        while (end < n && end - begin < kSmall && peer_of_slot_host[end] == p) ++end;
        if (end - begin == kSmall) end = std::upper_bound(peer_of_slot_host + end, peer_of_slot_host + n, p) - peer_of_slot_host;
        if (end - begin >= kSmall) place_peer<4>(begin, end, bits_host, stride, &bytes, place);
        else if (end > begin) place_peer<1>(begin, end, bits_host, stride, &bytes, place);
        begin = end;
    }
    peer_byte_ptr_out[n_peers] = bytes;
}

}  // namespace

extern "C" int adaqp_plan_layout(int64_t n, int32_t dim, const uint8_t *bits_host,
                                 const int32_t *peer_of_slot_host, int32_t n_peers, int64_t *perm_out,
                                 int64_t *row_offset_out, int64_t *peer_byte_ptr_out)
{
    if (n < 0 || dim <= 0 || n_peers < 0 || !peer_byte_ptr_out) return ADAQP_EINVAL;
    if (n > 0 && (!bits_host || !peer_of_slot_host || !perm_out || !row_offset_out)) return ADAQP_EINVAL;
    if (n > 0 && n_peers == 0) return ADAQP_EINVAL;
    ADAQP_TRY(check_slots(n, bits_host, peer_of_slot_host, n_peers));
    place_slots(n, dim, bits_host, peer_of_slot_host, n_peers, peer_byte_ptr_out, [&](int64_t i, int64_t k, int64_t byte) {
        perm_out[k] = i;
        row_offset_out[k] = byte;
    });
    return ADAQP_OK;
}

extern "C" int adaqp_plan_send(int64_t n, int32_t dim, const uint8_t *bits_host, const int32_t *peer_of_slot_host, int32_t n_peers,
                               const int32_t *send_idx_host, const int32_t *halo_idx_host, int64_t *perm_out, int64_t *row_offset_out,
                               int64_t *peer_byte_ptr_out, int32_t *send_idx_out, uint8_t *bits_out, int32_t *halo_idx_out,
                               int32_t *recv_order_out)
{
    if (n < 0 || dim <= 0 || n_peers < 0 || !peer_byte_ptr_out) return ADAQP_EINVAL;
    if (n > 0 && (!bits_host || !peer_of_slot_host || !perm_out || !row_offset_out || !send_idx_host || !send_idx_out || !bits_out)) return ADAQP_EINVAL;
    if (n > 0 && (n_peers == 0 || (halo_idx_host && (!halo_idx_out || !recv_order_out)))) return ADAQP_EINVAL;
    if (halo_idx_host && n > INT32_MAX) return ADAQP_ESIZE;
    ADAQP_TRY(check_slots(n, bits_host, peer_of_slot_host, n_peers));
    auto place = [&](int64_t i, int64_t k, int64_t byte) {
        perm_out[k] = i;
        row_offset_out[k] = byte;
        send_idx_out[k] = send_idx_host[i];
        bits_out[k] = bits_host[i];
    };
    if (!halo_idx_host || n == 0) {
        place_slots(n, dim, bits_host, peer_of_slot_host, n_peers, peer_byte_ptr_out, place);
        return ADAQP_OK;
    }
    // rows that ascend in the order of the slots (halo nodes numbered peer by peer): a slot's place is what the order lists
    bool ascending = true;
    for (int64_t i = 1; i < n; ++i) ascending &= halo_idx_host[i - 1] < halo_idx_host[i];
    place_slots(n, dim, bits_host, peer_of_slot_host, n_peers, peer_byte_ptr_out, [&](int64_t i, int64_t k, int64_t byte) {
        place(i, k, byte);
        halo_idx_out[k] = halo_idx_host[i];
        recv_order_out[i] = (int32_t)k;
    });
    if (!ascending) order_by_value(n, halo_idx_out, recv_order_out);
    return ADAQP_OK;
}

extern "C" int adaqp_plan_recv_order(int64_t n, const int32_t *halo_idx_host, int32_t *order_out)
{
    if (n < 0) return ADAQP_EINVAL;
    if (n == 0) return ADAQP_OK;
    if (!halo_idx_host || !order_out) return ADAQP_EINVAL;
    if (n > INT32_MAX) return ADAQP_ESIZE;
    order_by_value(n, halo_idx_host, order_out);
    return ADAQP_OK;
}

extern "C" int adaqp_plan_slot_of_row(int64_t n_rows, int64_t n, const int32_t *halo_idx_host,
                                      int32_t *slot_of_row_out)
{
    if (n_rows < 0 || n < 0) return ADAQP_EINVAL;
    if (n_rows > 0 && !slot_of_row_out) return ADAQP_EINVAL;
    if (n > 0 && !halo_idx_host) return ADAQP_EINVAL;
    if (n > INT32_MAX) return ADAQP_ESIZE;
    for (int64_t r = 0; r < n_rows; ++r) slot_of_row_out[r] = -1;
    for (int64_t t = 0; t < n; ++t) {
        const int32_t r = halo_idx_host[t];
        if (r < 0 || r >= n_rows || slot_of_row_out[r] != -1) return ADAQP_EINVAL;
        slot_of_row_out[r] = (int32_t)t;
    }
    return ADAQP_OK;
}

extern "C" int adaqp_plan_packed_rows(int64_t n_rows, int64_t n, const int32_t *halo_idx_host, const uint8_t *bits_host,
                                      const int64_t *row_offset_host, int32_t dim, int64_t packed_bytes, adaqp_packed_row *packed_row_out)
{
    if (n_rows < 0 || n < 0 || dim <= 0 || packed_bytes < 0 || (n_rows > 0 && !packed_row_out)) return ADAQP_EINVAL;
    if (n > 0 && (!halo_idx_host || !bits_host || !row_offset_host)) return ADAQP_EINVAL;
    if (n > INT32_MAX || packed_bytes >= (int64_t)kOutside) return ADAQP_ESIZE;
    std::fill_n(packed_row_out, n_rows, adaqp_packed_row{0, (uint32_t)n});          // a slot that there is not: not yet named
    for (int64_t t = 0; t < n; ++t) {
        const int32_t r = halo_idx_host[t];
        if (r < 0 || r >= n_rows || packed_row_out[r].slot != (uint32_t)n) return ADAQP_EINVAL;
        const int64_t stride = adaqp_row_stride(dim, bits_host[t]), at = row_offset_host[t];
        const bool ok = stride > 0 && at >= 0 && at % 4 == 0 && at + stride <= packed_bytes;
        packed_row_out[r] = ok ? adaqp_packed_row{(uint32_t)at | (bits_host[t] == 2 ? 1u : (bits_host[t] == 4 ? 2u : 3u)), (uint32_t)t}
                               : adaqp_packed_row{0, 0};
    }
    for (int64_t r = 0; r < n_rows; ++r)
        if (packed_row_out[r].place == 0) packed_row_out[r].slot = 0;
    return ADAQP_OK;
}

extern "C" int adaqp_plan_recv_segments(int64_t n, const int32_t *dst_idx_host, int32_t *order_out,
                                        int64_t *seg_ptr_out, int64_t *n_seg_out)
{
    if (n < 0 || !n_seg_out || !seg_ptr_out) return ADAQP_EINVAL;
    *n_seg_out = 0;
    seg_ptr_out[0] = 0;
    if (n == 0) return ADAQP_OK;
    if (!dst_idx_host || !order_out) return ADAQP_EINVAL;
    if (n > INT32_MAX) return ADAQP_ESIZE;
    order_by_value(n, dst_idx_host, order_out);
    int64_t n_seg = 0;
    int32_t before = 0;
    for (int64_t k = 0; k < n; ++k) {
        const int32_t dst = dst_idx_host[order_out[k]];
        if (k == 0 || dst != before) seg_ptr_out[n_seg++] = k;
        before = dst;
    }
    seg_ptr_out[n_seg] = n;
    *n_seg_out = n_seg;
    return ADAQP_OK;
}

namespace {

bool two_streams(const adaqp_layer_desc *d) { return d->schedule == ADAQP_ISOLATED || d->schedule == ADAQP_FREE; }

bool fused_receive(const adaqp_layer_desc *d)
{
    return d->direction == ADAQP_FORWARD && d->slot_of_row_dev && !d->tile_off_dependent_dev && d->n_send > 0 &&
           d->packed_bytes >= 4;
}

int check_desc(const adaqp_layer_desc *d)
{
    if (!d) return ADAQP_EINVAL;
    if (d->direction != ADAQP_FORWARD && d->direction != ADAQP_BACKWARD) return ADAQP_EINVAL;
    if (d->schedule < ADAQP_SERIAL || d->schedule > ADAQP_CHAIN) return ADAQP_EINVAL;
    if (d->dim <= 0 || d->ld < d->dim || d->ldo < d->dim || d->n_send < 0 || d->packed_bytes < 0 || d->nnz < 0)
        return ADAQP_EINVAL;
    if (d->overlap_begin < 0 || d->overlap_end < d->overlap_begin || d->dependent_begin < 0 ||
        d->dependent_end < d->dependent_begin)
        return ADAQP_EINVAL;
    // the two row ranges are written concurrently: they must not intersect
    if (d->overlap_begin < d->dependent_end && d->dependent_begin < d->overlap_end &&
        d->overlap_end > d->overlap_begin && d->dependent_end > d->dependent_begin)
        return ADAQP_EINVAL;
    if (!d->feat_dev || !d->out_dev || !d->rowptr_dev) return ADAQP_EINVAL;
    if (d->n_send > 0) {
        if (!d->send_idx_dev || !d->bits_dev || !d->row_offset_dev || !d->packed_dev || !d->params_dev ||
            !d->recv_packed_dev || !d->recv_params_dev)
            return ADAQP_EINVAL;
        if (d->direction == ADAQP_FORWARD && !d->halo_idx_dev) return ADAQP_EINVAL;
    }
    for (int part = 0; part < 2; ++part) {
        const adaqp_spmm_panels *p = part ? &d->panels_overlap : &d->panels_dependent;
        const int32_t *tile_off = part ? d->tile_off_overlap_dev : d->tile_off_dependent_dev;
        if (p->n_panels < 0 || p->n_per_tile < 0 || p->n_groups < 0 || p->n_panel_pieces < 0) return ADAQP_EINVAL;
        const adaqp_spmm_segments *s = part ? &d->segments_overlap : &d->segments_dependent;
        if (s->n_seg < 0 || s->n_entries < 0 || s->n_rows < 0) return ADAQP_EINVAL;
        if (s->n_seg > 0 && (!tile_off || !s->ptr_dev || !s->of_row_dev || !s->col_dev || !s->val_dev)) return ADAQP_EINVAL;
        const int64_t rb = part ? d->overlap_begin : d->dependent_begin, re = part ? d->overlap_end : d->dependent_end;
        const void *ws = part ? d->workspace_overlap_dev : d->workspace_dependent_dev;
        if (s->n_seg > 0) {
            if (s->n_rows != re - rb) return ADAQP_EINVAL;
            const int rc = check_segments_call(s, d->feat_dev, d->n_feat_rows, d->ld, d->dim, d->out_dev, d->ldo);
            if (rc != ADAQP_OK) return rc;
            if (re > rb && !aligned_to(ws, 256)) return ADAQP_EINVAL;
        }
        const adaqp_spmm_blocks *b = part ? &d->blocks_overlap : &d->blocks_dependent;
        if (b->n_blocks < 0 || b->n_pieces < 0 || b->n_steps < 0) return ADAQP_EINVAL;
        if (b->n_blocks > 0 && (!tile_off || p->n_panels > 0 || !b->rows_dev || !b->step_ptr_dev || !b->cols_dev || !b->table_dev))
            return ADAQP_EINVAL;
        if (b->n_blocks > 0) {
            const int rc = check_blocks_call(b, rb, re, d->feat_dev, d->n_feat_rows, d->ld, d->dim, d->out_dev, d->ldo);
            if (rc != ADAQP_OK) return rc;
            if (re > rb && !aligned_to(ws, 256)) return ADAQP_EINVAL;
        }
        if (p->n_panels == 0) continue;
        if (!tile_off) return ADAQP_EINVAL;                 // panels complement a tile table, never the merge path
        if (!p->panel_rows_dev || !p->pcol_dev || !p->palpha_dev || !p->piece_dev || !p->panel_piece_ptr_dev ||
            !p->panel_piece_dev)
            return ADAQP_EINVAL;
    }
    for (const adaqp_spmm_pieces *p : {&d->pieces_overlap, &d->pieces_dependent, &d->pieces_both}) {
        if (p->n_pieces == 0) continue;
        if (p->n_seg > INT32_MAX - 1024) return ADAQP_ESIZE;
        ADAQP_TRY(check_pieces(p, p->n_seg));
        if (d->overlap_end > d->overlap_begin && !aligned_to(d->workspace_overlap_dev, 256)) return ADAQP_EINVAL;
        if (d->dependent_end > d->dependent_begin && !aligned_to(d->workspace_dependent_dev, 256)) return ADAQP_EINVAL;
    }
    if (two_streams(d)) {
        if (!d->event_fork || !d->event_join) return ADAQP_EINVAL;
        if (d->stream_msg == d->stream_agg) return ADAQP_EINVAL;
        // the two aggregations run at the same time: they need separate scratch
        if (d->workspace_overlap_dev && d->workspace_overlap_dev == d->workspace_dependent_dev) return ADAQP_EINVAL;
    }
    return ADAQP_OK;
}

// Workspace of a row range: the partial sums of the tiled kernel or of the segments first, then (if the range has panels or blocks)
// the matrix-core kernel's piece sums, so that the two kernels can run at the same time.
int64_t tiled_part_bytes(const adaqp_layer_desc *d, bool overlap_part)
{
    const int64_t rows = overlap_part ? d->overlap_end - d->overlap_begin : d->dependent_end - d->dependent_begin;
    const adaqp_spmm_segments *seg = overlap_part ? &d->segments_overlap : &d->segments_dependent;
    int64_t bytes = 0;
    const int rc = seg->n_seg > 0 && seg->pieces.n_pieces > 0 ? adaqp_spmm_pieces_workspace_bytes(seg->pieces.n_partials, d->dim, &bytes)
                   : seg->n_seg > 0 ? adaqp_spmm_segments_workspace_bytes(seg->n_seg, seg->n_entries, d->dim, &bytes)
                                    : adaqp_spmm_tiled_workspace_bytes(rows, d->dim, &bytes);
    return rc == ADAQP_OK ? bytes : -1;
}

bool planned_for(const adaqp_spmm_pieces *p, int64_t rb, int64_t re)
{
    return p->n_pieces > 0 && re > rb && p->n_seg == re - rb && p->row_begin == rb;
}

// Whether rows [rb, re) go as planned; fused: with received rows read from the receive buffer.  Matrices of another layout than the one
// that the kernels of the plan are built for, or too large for it, go along the merge path as without a plan.
bool takes_pieces(const adaqp_layer_desc *d, const adaqp_spmm_pieces *pieces, int64_t rb, int64_t re, bool fused)
{
    if (!planned_for(pieces, rb, re)) return false;
    if (d->ld % 32 != 0 || d->ldo % 32 != 0 || !aligned_to(d->feat_dev, 128) || !aligned_to(d->out_dev, 128)) return false;
    if (!d->col_dev || !d->val_dev || !aligned_to(d->rowptr_dev, 8) || !aligned_to(d->col_dev, 4) || !aligned_to(d->val_dev, 4)) return false;
    if (fused && (!d->packed_row_dev || !aligned_to(d->slot_of_row_dev, 4) || !aligned_to(d->recv_packed_dev, 4) ||
                  !aligned_to(d->recv_params_dev, 8) || !aligned_to(d->row_offset_dev, 8) || !aligned_to(d->packed_row_dev, 8)))
        return false;
    return sliced_takes(re - rb, d->nnz, d->n_feat_rows, d->ld, fused, d->packed_bytes, d->dim);
}

// Workspace of rows [rb, re) without tiles, whether planned or not.
int range_bytes(const adaqp_layer_desc *d, const adaqp_spmm_pieces *pieces, int64_t rb, int64_t re, int64_t nz, bool fused, int64_t *bytes)
{
    ADAQP_TRY(adaqp_spmm_workspace_bytes(re - rb, nz, d->dim, bytes));
    if (!takes_pieces(d, pieces, rb, re, fused)) return ADAQP_OK;
    int64_t planned = 0;
    ADAQP_TRY(adaqp_spmm_pieces_workspace_bytes(pieces->n_partials, d->dim, &planned));
    *bytes = std::max(*bytes, planned);
    return ADAQP_OK;
}

// Whether the memory that is sent is no part of b.
bool send_buffers_apart(const adaqp_layer_desc *d, const void *b, int64_t b_bytes)
{
    auto apart = [&](const void *a, int64_t a_bytes) {
        const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
        return !a || !b || x + (uint64_t)a_bytes <= y || y + (uint64_t)b_bytes <= x;
    };
    return apart(d->packed_dev, d->packed_bytes) && apart(d->params_dev, d->n_send * 2 * (int64_t)sizeof(float));
}

// CHAIN has nothing to overlap the transfer with, and the copy that stands in for it is a launch of 2.5 to 5 us that leaves the GPU part
// empty.  There the launch that receives takes the bytes from where the copy takes them, and copies them beside; the table of received
// rows is then filled in the quantisation's launch.  An exchange with another GPU would have to end before its receive begins: what this saves
// it saves in the loop-back only.  Whole steps, launch by launch in turn: 2 000 rows, 128 columns 15.1 -> 13.0 us, 24 000 rows, 66 columns, packed
// 30.1 -> 27.6, 306 000 rows, 256 columns 754.6 -> 751.6, 179 000 rows, 300 columns 345.6 -> 341.0, 30 000 nodes backward 104.6 -> 102.2.
// Buffers that the receiving calls refuse go the other way, and are refused there.  So do send buffers in memory that the launch writes, which
// a caller may use again once the messages are on their way: rows of feat that are received, out, a workspace.
bool receives_beside(const adaqp_layer_desc *d)
{
    if (!(d->schedule == ADAQP_CHAIN && d->n_send > 0 && d->n_send < kBesideMessages && d->packed_bytes >= 4 && aligned_to(d->packed_dev, 4) &&
          aligned_to(d->params_dev, 8) && aligned_to(d->recv_packed_dev, 4) && aligned_to(d->recv_params_dev, 8)))
        return false;
    return send_buffers_apart(d, d->feat_dev, d->n_feat_rows * d->ld * (int64_t)sizeof(float)) &&
           send_buffers_apart(d, d->out_dev, std::max(d->overlap_end, d->dependent_end) * d->ldo * (int64_t)sizeof(float)) &&
           send_buffers_apart(d, d->workspace_overlap_dev, d->workspace_overlap_bytes) &&
           send_buffers_apart(d, d->workspace_dependent_dev, d->workspace_dependent_bytes);
}

// Rows [rb, re) as planned, or along the merge path; fused: received rows are read from the receive buffer.
int aggregate_range(const adaqp_layer_desc *d, int64_t rb, int64_t re, int64_t nz, bool fused, const adaqp_spmm_pieces *pieces, void *ws,
                    int64_t wsb, hipStream_t st)
{
    if (takes_pieces(d, pieces, rb, re, fused)) {
        PieceArgs a = {};
        a.ptr = d->rowptr_dev + rb;
        a.col = d->col_dev;
        a.val = d->val_dev;
        a.n_entries = d->nnz;
        a.n_walked = nz;
        a.n_seg = a.n_rows = (int32_t)(re - rb);
        a.of_rows = true;
        a.H = d->feat_dev;
        a.n_cols = d->n_feat_rows;
        a.ldh = d->ld;
        if (fused) {
            const bool beside = receives_beside(d);
            a.p = PackedRows{d->slot_of_row_dev, beside ? d->packed_dev : d->recv_packed_dev, d->packed_bytes,
                             beside ? d->params_dev : d->recv_params_dev, d->bits_dev, d->row_offset_dev, d->n_send, 0, d->dim, d->packed_row_dev};
            a.copies = beside ? loop_back_of(d) : kNoLoopBack;
        }
        a.dim = d->dim;
        a.out = d->out_dev + rb * d->ldo;
        a.ldo = d->ldo;
        a.partial = static_cast<float *>(ws);
        return launch_pieces(pieces, a, st);
    }
    return spmm_rows(d->rowptr_dev, d->col_dev, d->val_dev, d->nnz, rb, re, nz, d->feat_dev, d->n_feat_rows, d->ld, d->dim,
                     d->out_dev, d->ldo, fused ? d->slot_of_row_dev : nullptr, d->recv_packed_dev, d->packed_bytes,
                     d->recv_params_dev, d->bits_dev, d->row_offset_dev, d->n_send, ws, wsb, st,
                     d->direction == ADAQP_BACKWARD);
}

// The rows of a range that are aggregated entry by entry: all of them, or those outside the panels.
int aggregate_rows(const adaqp_layer_desc *d, bool overlap_part, hipStream_t st)
{
    const int64_t rb = overlap_part ? d->overlap_begin : d->dependent_begin;
    const int64_t re = overlap_part ? d->overlap_end : d->dependent_end;
    const int64_t nz = overlap_part ? d->overlap_nnz : d->dependent_nnz;
    void *ws = overlap_part ? d->workspace_overlap_dev : d->workspace_dependent_dev;
    const int64_t wsb = overlap_part ? d->workspace_overlap_bytes : d->workspace_dependent_bytes;
    const int32_t *tile_off = overlap_part ? d->tile_off_overlap_dev : d->tile_off_dependent_dev;
    const adaqp_spmm_segments *seg = overlap_part ? &d->segments_overlap : &d->segments_dependent;
    if (tile_off && seg->n_seg > 0)
        return adaqp_spmm_csr_segments(seg, d->feat_dev, d->n_feat_rows, d->ld, d->dim, d->out_dev + rb * d->ldo, d->ldo, ws, wsb, st);
    if (tile_off)
        return adaqp_spmm_csr_tiled(d->rowptr_dev, d->col_dev, d->val_dev, d->nnz, rb, re, d->feat_dev,
                                    d->n_feat_rows, d->ld, d->dim, d->out_dev, d->ldo, tile_off,
                                    overlap_part ? d->tile_chunk_overlap : d->tile_chunk_dependent, ws, wsb, st);
    return aggregate_range(d, rb, re, nz, !overlap_part && fused_receive(d), overlap_part ? &d->pieces_overlap : &d->pieces_dependent, ws,
                           wsb, st);
}

bool has_blocks(const adaqp_layer_desc *d, bool overlap_part)
{
    const int32_t *tile_off = overlap_part ? d->tile_off_overlap_dev : d->tile_off_dependent_dev;
    return tile_off && (overlap_part ? d->blocks_overlap.n_blocks : d->blocks_dependent.n_blocks) > 0;
}

// Panels or blocks: rows that a matrix-core kernel takes.
bool has_panels(const adaqp_layer_desc *d, bool overlap_part)
{
    const int32_t *tile_off = overlap_part ? d->tile_off_overlap_dev : d->tile_off_dependent_dev;
    return tile_off && ((overlap_part ? d->panels_overlap.n_panels : d->panels_dependent.n_panels) > 0 || has_blocks(d, overlap_part));
}

// The rows of a range that were struck from its tile table.  Own part of the workspace, disjoint output rows:
// independent of aggregate_rows of the same range.
int aggregate_panels(const adaqp_layer_desc *d, bool overlap_part, hipStream_t st)
{
    if (!has_panels(d, overlap_part)) return ADAQP_OK;
    const int64_t rb = overlap_part ? d->overlap_begin : d->dependent_begin;
    const int64_t re = overlap_part ? d->overlap_end : d->dependent_end;
    char *ws = static_cast<char *>(overlap_part ? d->workspace_overlap_dev : d->workspace_dependent_dev);
    const int64_t wsb = overlap_part ? d->workspace_overlap_bytes : d->workspace_dependent_bytes;
    const int64_t skip = tiled_part_bytes(d, overlap_part);
    if (skip < 0 || !ws || wsb < skip) return ADAQP_ESIZE;
    if (has_blocks(d, overlap_part))
        return adaqp_spmm_csr_blocks(overlap_part ? &d->blocks_overlap : &d->blocks_dependent, rb, re, d->feat_dev,
                                     d->n_feat_rows, d->ld, d->dim, d->out_dev, d->ldo, ws + skip, wsb - skip, st);
    return adaqp_spmm_csr_panels(overlap_part ? &d->panels_overlap : &d->panels_dependent, rb, re, d->feat_dev,
                                 d->n_feat_rows, d->ld, d->dim, d->out_dev, d->ldo, ws + skip, wsb - skip, st);
}

int aggregate(const adaqp_layer_desc *d, bool overlap_part, hipStream_t st)
{
    const int rc = aggregate_rows(d, overlap_part, st);
    return rc != ADAQP_OK ? rc : aggregate_panels(d, overlap_part, st);
}

// The table of received rows is filled beside the copies, which do not fill the GPU (34 000 rows, 66 columns, the whole step: 35.1 us, 35.0 with
// a table that the host made).
__global__ __launch_bounds__(kBlock) void loop_back_kernel(const LoopBack c, const PackedRowArgs p)
{
    const uint32_t copying = c.blocks_packed + c.blocks_params;
    if (blockIdx.x >= copying) fill_packed_rows(p, blockIdx.x - copying);
    else copy_blocks(c, blockIdx.x, kBlock);
}

int loop_back(const adaqp_layer_desc *d, bool fill_table, hipStream_t st)
{
    if (d->n_send == 0) return ADAQP_OK;
    const LoopBack c = loop_back_of(d);
    const PackedRowArgs p = fill_table ? packed_rows_of(d) : kNoPackedRows;
    hipLaunchKernelGGL(loop_back_kernel, dim3(c.blocks() + p.blocks), dim3(kBlock), 0, st, c, p);
    ADAQP_HIP_TRY(hipGetLastError());
    return ADAQP_OK;
}

int64_t range_nnz(const adaqp_layer_desc *d, bool overlap_part)
{
    const int64_t nz = overlap_part ? d->overlap_nnz : d->dependent_nnz;
    return nz < 0 || nz > d->nnz ? d->nnz : nz;
}

int64_t both_nnz(const adaqp_layer_desc *d) { return std::min(range_nnz(d, true) + range_nnz(d, false), d->nnz); }

bool larger_is_overlap(const adaqp_layer_desc *d) { return d->workspace_overlap_bytes >= d->workspace_dependent_bytes; }

// CHAIN: both row ranges in one launch, if neither has tiles, they are neighbours and one of the workspaces can take them.  A
// second aggregation is two launches and another start and end on a part empty GPU (SERIAL against CHAIN: 2 000 rows 45 us,
// 27; 24 000 rows 58, 42; 50 000-row backward step 120, 108; 179 000 rows 425, 419).
bool one_launch(const adaqp_layer_desc *d)
{
    if (d->schedule != ADAQP_CHAIN || d->tile_off_overlap_dev || d->tile_off_dependent_dev) return false;
    if (d->overlap_end != d->dependent_begin || d->overlap_end == d->overlap_begin || d->dependent_end == d->dependent_begin)
        return false;
    const int64_t rows = d->dependent_end - d->overlap_begin;
    int64_t need = 0;
    if (rows > INT32_MAX - 1) return false;
    if (range_bytes(d, &d->pieces_both, d->overlap_begin, d->dependent_end, both_nnz(d), fused_receive(d), &need) != ADAQP_OK) return false;
    return larger_is_overlap(d) ? d->workspace_overlap_dev && d->workspace_overlap_bytes >= need
                                : d->workspace_dependent_dev && d->workspace_dependent_bytes >= need;
}

// With the received rows still packed the launch looks a slot up for every column, also those of rows that cannot have one: a
// step that de-quantises first must give the same bits, so it has to be cut the same way.
int aggregate_both(const adaqp_layer_desc *d, hipStream_t st)
{
    const bool first = larger_is_overlap(d);
    return aggregate_range(d, d->overlap_begin, d->dependent_end, both_nnz(d), fused_receive(d), &d->pieces_both,
                           first ? d->workspace_overlap_dev : d->workspace_dependent_dev,
                           first ? d->workspace_overlap_bytes : d->workspace_dependent_bytes, st);
}

int quantise(const adaqp_layer_desc *d, bool fill_table, hipStream_t st)
{
    const bool forward = d->direction == ADAQP_FORWARD;
    return quantize_pack_beside(forward ? d->feat_dev : d->out_dev, forward ? d->n_feat_rows : std::max(d->dependent_end, d->overlap_end),
                                forward ? d->ld : d->ldo, d->dim, d->send_idx_dev, d->bits_dev, d->row_offset_dev, d->n_send, d->seed,
                                d->packed_dev, d->packed_bytes, d->params_dev, d->alpha_sq_dev, d->beta_dev,
                                fill_table ? packed_rows_of(d) : kNoPackedRows, st);
}

// Whether received messages become additions to rows of out.
bool adds_received(const adaqp_layer_desc *d)
{
    return d->direction == ADAQP_BACKWARD && d->n_recv_seg > 0 && d->recv_seg_order_dev && d->recv_seg_ptr_dev && d->halo_idx_dev;
}

// What the received messages become: halo rows of feat (forward, unless the aggregation reads them packed), or additions
// to rows of out (backward, if segments are given).  beside: the loop-back copy is part of the launch.
int receive(const adaqp_layer_desc *d, bool beside, hipStream_t st)
{
    const uint8_t *packed = beside ? d->packed_dev : d->recv_packed_dev;
    const float *params = beside ? d->params_dev : d->recv_params_dev;
    const LoopBack copies = beside ? loop_back_of(d) : kNoLoopBack;
    if (d->direction == ADAQP_FORWARD) {
        if (fused_receive(d)) return ADAQP_OK;
        return unpack_dequant_beside(packed, d->packed_bytes, params, d->bits_dev, d->row_offset_dev, d->halo_idx_dev, d->recv_order_dev,
                                     d->n_send, d->dim, d->feat_dev, d->n_feat_rows, d->ld, copies, st);
    }
    if (!adds_received(d)) return ADAQP_OK;
    return unpack_dequant_add_beside(packed, d->packed_bytes, params, d->bits_dev, d->row_offset_dev, d->halo_idx_dev, d->n_send,
                                     d->recv_seg_order_dev, d->recv_seg_ptr_dev, d->n_recv_seg, d->dim, d->out_dev,
                                     std::max(d->dependent_end, d->overlap_end), d->ldo, copies, st);
}

}  // namespace

extern "C" int64_t adaqp_layer_desc_bytes(void) { return (int64_t)sizeof(adaqp_layer_desc); }

extern "C" int adaqp_layer_step(const adaqp_layer_desc *d)
{
    int rc = check_desc(d);
    if (rc != ADAQP_OK) return rc;
    // workspace sizes are checked up front so that a failure cannot leave the two streams half-joined
    for (int part = 0; part < 2; ++part) {
        const int64_t rows = part ? d->overlap_end - d->overlap_begin : d->dependent_end - d->dependent_begin;
        int64_t nz = part ? d->overlap_nnz : d->dependent_nnz;
        if (nz < 0 || nz > d->nnz) nz = d->nnz;
        int64_t need = 0;
        rc = range_bytes(d, part ? &d->pieces_overlap : &d->pieces_dependent, part ? d->overlap_begin : d->dependent_begin,
                         part ? d->overlap_end : d->dependent_end, nz, part == 0 && fused_receive(d), &need);
        if (rc != ADAQP_OK) return rc;
        if (part ? d->tile_off_overlap_dev != nullptr : d->tile_off_dependent_dev != nullptr) {
            need = tiled_part_bytes(d, part != 0);          // that range takes the tiled kernel, or its segments
            if (need < 0) return ADAQP_ESIZE;
            const adaqp_spmm_panels *panels = part ? &d->panels_overlap : &d->panels_dependent;
            if (panels->n_panels > 0) {
                int64_t need_panels = 0;
                rc = adaqp_spmm_panels_workspace_bytes(panels->n_per_tile, d->dim, &need_panels);
                if (rc != ADAQP_OK) return rc;
                need += need_panels;                        // side by side: the two kernels may run together
            }
            const adaqp_spmm_blocks *blocks = part ? &d->blocks_overlap : &d->blocks_dependent;
            if (blocks->n_blocks > 0) {
                int64_t need_blocks = 0;
                rc = adaqp_spmm_blocks_workspace_bytes(blocks->n_blocks, blocks->n_pieces, d->dim, &need_blocks);
                if (rc != ADAQP_OK) return rc;
                need += need_blocks;
            }
        }
        const int64_t have = part ? d->workspace_overlap_bytes : d->workspace_dependent_bytes;
        const void *ws = part ? d->workspace_overlap_dev : d->workspace_dependent_dev;
        if (rows > 0 && need > 0 && (!ws || have < need)) return ADAQP_ESIZE;
    }

    hipStream_t msg = (hipStream_t)d->stream_msg;
    hipStream_t agg = two_streams(d) ? (hipStream_t)d->stream_agg : msg;
    hipEvent_t fork = (hipEvent_t)d->event_fork, join = (hipEvent_t)d->event_join;
    const bool forward = d->direction == ADAQP_FORWARD;
    const bool both_tiled = d->tile_off_overlap_dev && d->tile_off_dependent_dev;
    const bool joint = one_launch(d);
    const bool paired = forward && both_tiled && two_streams(d) &&
                        (has_panels(d, true) || has_panels(d, false));
    const bool fills = fused_receive(d) && takes_pieces(d, joint ? &d->pieces_both : &d->pieces_dependent,
                                                        joint ? d->overlap_begin : d->dependent_begin, d->dependent_end, true);
    // whether there is a launch that takes the loop-back copy with it
    const bool beside = receives_beside(d) && (forward ? !fused_receive(d) || fills : adds_received(d) && d->n_recv_seg <= d->n_send);
    bool forked = false;
    auto fork_now = [&]() -> int {
        if (!two_streams(d)) return ADAQP_OK;
        ADAQP_HIP_TRY(hipEventRecord(fork, msg));
        ADAQP_HIP_TRY(hipStreamWaitEvent(agg, fork, 0));
        forked = true;
        return ADAQP_OK;
    };
    auto join_now = [&]() -> int {
        if (!forked) return ADAQP_OK;
        ADAQP_HIP_TRY(hipEventRecord(join, agg));
        ADAQP_HIP_TRY(hipStreamWaitEvent(msg, join, 0));
        forked = false;
        return ADAQP_OK;
    };
    auto agg_waits_for_msg = [&]() -> int {
        // the fork event is free again: its first wait has been enqueued, and a wait refers to the record before it
        ADAQP_HIP_TRY(hipEventRecord(fork, msg));
        ADAQP_HIP_TRY(hipStreamWaitEvent(agg, fork, 0));
        return ADAQP_OK;
    };
#define ADAQP_STEP(expr)                    \
    do {                                    \
        rc = (expr);                        \
        if (rc != ADAQP_OK) { join_now(); return rc; } \
    } while (0)

    if (forward) {
        // FREE: the central rows start right away.  ISOLATED: they start once quantisation is done.
        if (d->schedule == ADAQP_FREE) {
            ADAQP_STEP(fork_now());
            ADAQP_STEP(paired ? aggregate_rows(d, true, agg) : aggregate(d, true, agg));
        }
        ADAQP_STEP(quantise(d, fills && beside, msg));
        if (d->schedule == ADAQP_ISOLATED) {
            ADAQP_STEP(fork_now());
            ADAQP_STEP(paired ? aggregate_rows(d, true, agg) : aggregate(d, true, agg));
        }
        if (!beside) ADAQP_STEP(loop_back(d, fills, msg));
        ADAQP_STEP(receive(d, beside, msg));
        if (!two_streams(d) && !joint) ADAQP_STEP(aggregate(d, true, msg));
        if (joint) {
            ADAQP_STEP(aggregate_both(d, msg));
        } else if (paired) {
            // a panel kernel (matrix cores) and a tiled kernel (vector-memory pipeline) fill each other's gaps:
            // both tiled launches on the second stream, one after the other, both panel launches here
            ADAQP_STEP(agg_waits_for_msg());                            // the halo rows are in place
            ADAQP_STEP(aggregate_panels(d, true, msg));
            ADAQP_STEP(aggregate_rows(d, false, agg));
            ADAQP_STEP(aggregate_panels(d, false, msg));
        } else {
            // two tiled aggregations side by side would bring two column ranges to every L2 and lose what the
            // tiling is for: the dependent one waits for the other (which has overlapped the message path by now)
            if (both_tiled) ADAQP_STEP(join_now());
            ADAQP_STEP(aggregate(d, false, msg));
        }
    } else {
        // backward: the rows that are sent are aggregated first, the local rows overlap their quantisation
        // (FREE) or only their transfer (ISOLATED)
        if (d->schedule == ADAQP_FREE) {
            ADAQP_STEP(fork_now());
            ADAQP_STEP(aggregate(d, true, agg));
            if (both_tiled) ADAQP_STEP(join_now());         // as in the forward step: one tiled launch at a time
        }
        ADAQP_STEP(joint ? aggregate_both(d, msg) : aggregate(d, false, msg));
        ADAQP_STEP(quantise(d, fills && beside, msg));
        if (d->schedule == ADAQP_ISOLATED) {
            ADAQP_STEP(fork_now());
            ADAQP_STEP(aggregate(d, true, agg));
        }
        if (!beside) ADAQP_STEP(loop_back(d, fills, msg));
        if (!two_streams(d) && !joint) ADAQP_STEP(aggregate(d, true, msg));
        // the received gradients are added to rows that the local aggregation also writes: join first
        ADAQP_STEP(join_now());
        ADAQP_STEP(receive(d, beside, msg));
    }
    ADAQP_STEP(join_now());
#undef ADAQP_STEP
    return ADAQP_OK;
}
