"""Device-resident state of one partition's layer step: uploads a partition, plans the buffer layout,
allocates buffers / workspaces / streams / events with torch and HIP, and fills an adaqp_layer_desc.

Everything computational happens inside libadaqp; this module only owns memory and handles.
"""
from __future__ import annotations

import ctypes
import weakref
from typing import Optional

import numpy as np
import torch

from . import binding as B
from .synth import Partition, alpha_sq_stand_in

# What a second stream can hide is the transfer: the loop-back copy of this many bytes takes about 25 us.  Its price is a fork and
# a join (about 25 us), a second aggregation, and two gathers that compete for the L2s and what is behind them (ISOLATED
# against CHAIN: 2 000 rows 42 us, 27; 24 000 rows 64, 42; 50 000-row backward step 141, 108; 179 000 rows 435, 419).
CHAIN_BYTES = 64 << 20

_hip: Optional[ctypes.CDLL] = None


def _hip_runtime() -> ctypes.CDLL:
    global _hip
    if _hip is None:
        _hip = ctypes.CDLL("libamdhip64.so")
        _hip.hipEventCreateWithFlags.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint]
        _hip.hipEventCreateWithFlags.restype = ctypes.c_int
        _hip.hipEventDestroy.argtypes = [ctypes.c_void_p]
        _hip.hipEventDestroy.restype = ctypes.c_int
        _hip.hipStreamIsCapturing.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_int)]
        _hip.hipStreamIsCapturing.restype = ctypes.c_int
    return _hip


def _capturing(stream: torch.cuda.Stream) -> bool:
    """torch answers this for the current stream only, and making another one current costs every step 10 us and more."""
    status = ctypes.c_int(0)
    rc = _hip_runtime().hipStreamIsCapturing(stream.cuda_stream, ctypes.byref(status))
    if rc != 0:
        raise RuntimeError(f"hipStreamIsCapturing failed: {rc}")
    return status.value != 0


class HipEvent:
    """A raw hipEvent_t (timing disabled) whose handle can be passed through the C ABI."""
    _DISABLE_TIMING = 0x2

    def __init__(self):
        h = ctypes.c_void_p()
        rc = _hip_runtime().hipEventCreateWithFlags(ctypes.byref(h), self._DISABLE_TIMING)
        if rc != 0:
            raise RuntimeError(f"hipEventCreateWithFlags failed: {rc}")
        self.handle = h.value

    def __del__(self):
        try:
            if getattr(self, "handle", None):
                _hip_runtime().hipEventDestroy(self.handle)
        except Exception:
            pass


class SendPlan:
    """Sorted slot order and byte offsets of one direction's messages (host arrays + device copies)."""

    def __init__(self, dim: int, send_idx: np.ndarray, bits: np.ndarray, peer_of_slot: np.ndarray,
                 n_peers: int, halo_idx: Optional[np.ndarray], device, add_segments: bool = False):
        # one pass over the slots for all arrays, and one upload: 100 000 slots 622 -> 321 us
        plan = B.adaqp_plan_send(dim, bits, peer_of_slot, n_peers, send_idx, None if halo_idx is None or halo_idx.size == 0 else halo_idx)
        self.perm, self.row_offset_host, self.peer_byte_ptr = plan["perm"], plan["row_offset"], plan["peer_byte_ptr"]
        self.send_idx_host, self.bits_host = plan["send_idx"], plan["bits"]
        self.halo_idx_host, self.recv_order_host = plan.get("halo_idx"), plan.get("recv_order")
        self.n = int(self.perm.shape[0])
        self.packed_bytes = int(self.peer_byte_ptr[-1])
        blob = torch.from_numpy(plan["blob"]).to(device)
        on_device = {name: blob[begin:begin + size].view(torch.from_numpy(plan[name]).dtype) for name, (begin, size, _) in plan["at"].items()}
        self.send_idx, self.bits, self.row_offset = on_device["send_idx"], on_device["bits"], on_device["row_offset"]
        self.halo_idx, self.recv_order = on_device.get("halo_idx"), on_device.get("recv_order")
        # backward receive: slots grouped by destination row
        self.seg_order = self.seg_ptr = None
        if add_segments and self.halo_idx_host is not None:
            order, seg_ptr = B.adaqp_plan_recv_segments(self.halo_idx_host)
            self.seg_order_host, self.seg_ptr_host = order, seg_ptr
            self.seg_order = torch.from_numpy(order).to(device)
            self.seg_ptr = torch.from_numpy(seg_ptr).to(device)


def line_padded(a: np.ndarray, device, pad: bool = True, spread: bool = False) -> torch.Tensor:
    """Uploads a [n, dim] fp32 matrix into rows whose pitch is a whole number of 128-byte lines (the layout
    the kernels are built for) and returns the [n, dim] view; the padding columns are zero.  With `spread` the number of
    lines is never a multiple of four: an aggregation that takes the same lines of every row would find them in a quarter of
    the L1's sets or fewer (256 columns, transposed graph: 0.84 ms at a pitch of 8 lines, 0.80 at 9)."""
    n, dim = a.shape
    ld = dim
    if pad:
        lines = (dim + 31) // 32
        ld = 32 * (lines + 1 if spread and lines % 4 == 0 else lines)
    buf = torch.zeros((n, ld), dtype=torch.float32, device=device)
    view = buf[:, :dim]
    view.copy_(torch.from_numpy(a))
    return view


def _or_none(plan, *args, **options):
    """What plan(*args) returns, or None where the library refuses the rows, there would be too many pieces, or there is no room to plan
    them.  Pieces are never needed: the walk is cut on the device then, by kernels that take any rows."""
    try:
        return plan(*args, **options)
    except MemoryError:
        return None
    except B.AdaqpError as e:
        if e.status not in (B.EINVAL, B.ESIZE):
            raise
        return None


class LayerStep:
    def __init__(self, p: Partition, device="cuda:0", seed: int = 0, pad: bool = True, use_recv_order: bool = False,
                 backward_receive: bool = True, trace: bool = True, fused_receive: bool = False,
                 tiled: Optional[bool] = None, panels: Optional[bool] = None, panel_min_row=B.SPMM_PANEL_MIN_ROW,
                 panel_piece_cols: int = B.SPMM_PANEL_PIECE_COLS, streams=None):
        self.p = p
        self.device = torch.device(device)
        dev = self.device
        cfg = p.cfg
        self.dim = cfg.dim
        self.backward = bool(cfg.backward)
        self.seed = seed
        self.use_recv_order = use_recv_order
        self.backward_receive = backward_receive
        self.fused_receive = fused_receive and not self.backward
        self.col = torch.from_numpy(p.col).to(dev)
        with torch.inference_mode(False):           # a tensor made in inference mode does not count what is written to it
            self.rowptr = torch.from_numpy(p.rowptr).to(dev)
            self.val = torch.from_numpy(p.val).to(dev)
        self.feat = line_padded(p.feat, dev, pad, spread=True)
        self.out = line_padded(np.zeros((p.n_rows, cfg.dim), dtype=np.float32), dev, pad, spread=True)
        self.plan = SendPlan(cfg.dim, p.send_idx, p.bits, p.peer_of_slot, cfg.n_peers, p.halo_idx, dev,
                             add_segments=self.backward)
        n = self.plan.n
        # forward, fused receive: the dependent aggregation reads received rows straight from the receive buffer
        self.slot_of_row = self.packed_row = None
        self._unplanned_dependent = None
        self.set_fused_receive(self.fused_receive)
        nbytes = max(self.plan.packed_bytes, 4)
        self.packed = torch.zeros(nbytes, dtype=torch.uint8, device=dev)
        self.params = torch.zeros((max(n, 1), 2), dtype=torch.float32, device=dev)
        # trace for the bit-width assigner: per slot, the sum of squared coefficients the message meets on its
        # target device is an input (the generator supplies a stand-in)
        self.alpha_sq = self.beta = None
        if trace and n > 0:
            self.alpha_sq_host = np.ascontiguousarray(alpha_sq_stand_in(p)[self.plan.perm])
            self.alpha_sq = torch.from_numpy(self.alpha_sq_host).to(dev)
            self.beta = torch.zeros(n, dtype=torch.float32, device=dev)
        self.recv_packed = torch.zeros(nbytes, dtype=torch.uint8, device=dev)
        self.recv_params = torch.zeros((max(n, 1), 2), dtype=torch.float32, device=dev)
        ob, oe = p.overlap_rows
        db, de = p.dependent_rows
        self.overlap_nnz = int(p.rowptr[oe] - p.rowptr[ob])
        self.dependent_nnz = int(p.rowptr[de] - p.rowptr[db])
        # aggregation tiled over the L2 caches: pays when rows are long (every row of feat re-used many times).
        # tiled=None lets the library decide: by what segments of both ranges save, or where they cannot be used per
        # row range (adaqp_spmm_tiled_pays: mean row length).
        self._lines = {}                            # per slice of pieces, of ranges that the rule has been asked about
        self.tile_off_overlap = self.tile_off_dependent = None
        self.tile_chunk_overlap = self.tile_chunk_dependent = 0
        self._tiles_asked_for = tiled
        # within a tiled range, rows that list a good part of the columns go to the matrix cores: panels=None in dense blocks,
        # where the library says that pays (tiled=True: where they can be more than a few workgroups); True: rows of panel_min_row entries in panels, always
        self.panels_overlap = self.panels_dependent = B.DevicePanels(None)
        self.blocks_overlap = self.blocks_dependent = B.DeviceBlocks(None)
        # and the others' entries are kept a second time, in the order of the tiles
        self.segments_overlap = self.segments_dependent = B.DeviceSegments(None)
        # panel_min_row: one threshold, or one per row range (overlap, dependent)
        min_row_o, min_row_d = panel_min_row if isinstance(panel_min_row, tuple) else (panel_min_row, panel_min_row)
        ws_o = B.adaqp_spmm_workspace_bytes(oe - ob, self.overlap_nnz, cfg.dim)
        ws_d = B.adaqp_spmm_workspace_bytes(de - db, self.dependent_nnz, cfg.dim)
        if oe == db:        # CHAIN aggregates both ranges in one launch, if this workspace can take them
            ws_o = max(ws_o, B.adaqp_spmm_workspace_bytes(de - ob, self.overlap_nnz + self.dependent_nnz, cfg.dim))
        if pad and tiled is not False:
            plan_dependent = (panels, min_row_d, panel_piece_cols)
            if self.fused_receive:
                # tiles do not read received rows that stay packed: planned when they are to be de-quantised first
                tile_overlap, tile_dependent = self._ranges_to_tile(tiled, p.overlap_rows)[0], False
                self._unplanned_dependent = (tiled, *plan_dependent)
            else:
                tile_overlap, tile_dependent = self._ranges_to_tile(tiled, p.overlap_rows, p.dependent_rows)
            if tile_overlap:
                (self.tile_off_overlap, self.tile_chunk_overlap, self.panels_overlap, self.blocks_overlap, self.segments_overlap,
                 need) = self._plan_long_rows(ob, oe, panels, min_row_o, panel_piece_cols)
                ws_o = max(ws_o, need)
            if tile_dependent:
                ws_d = max(ws_d, self._plan_dependent(*plan_dependent))
        self._plan_rows(pad)
        ws_o, ws_d = max(ws_o, self._pieces_bytes(self.pieces_overlap)), max(ws_d, self._pieces_bytes(self.pieces_dependent))
        if self.pieces_both:
            ws_o = max(ws_o, self._pieces_bytes(self.pieces_both))
        self.ws_overlap = torch.empty(max(ws_o, 256), dtype=torch.uint8, device=dev)
        self.ws_dependent = torch.empty(max(ws_d, 256), dtype=torch.uint8, device=dev)
        # streams=(msg, agg): take over an existing pair.  HIP deals streams to a few hardware queues in turn, so a
        # process that keeps creating streams can end up with a step's two streams on one queue (no overlap)
        self.stream_msg, self.stream_agg = streams if streams is not None else (torch.cuda.Stream(device=dev),
                                                                                  torch.cuda.Stream(device=dev))
        # the tables of blocks and segments hold the coefficients a second time; kernels write them
        self._copied = self._coefficients()
        self._captured = []                         # what val was in captures, whose replays copy it
        self._order_copies()
        self.event_fork = HipEvent()
        self.event_join = HipEvent()

    def _plan_rows(self, pad: bool) -> None:
        """Pieces of the walk over the rows of ranges without tiles."""
        p, none = self.p, B.DevicePieces(None)
        self.pieces_overlap = self.pieces_dependent = self.pieces_both = none
        self._planned_rows = self._rows_tensor()
        n_cols = p.feat.shape[0]
        if not pad or p.nnz == 0 or n_cols * self.feat.stride(0) * 4 >= B.SPMM_SEGMENTS_MOST_BYTES:
            return
        (ob, oe), (db, de) = p.overlap_rows, p.dependent_rows
        plain = [r for r, tiles in (((ob, oe), self.tile_off_overlap), ((db, de), self.tile_off_dependent)) if r[1] > r[0] and tiles is None]
        if not plain:
            return
        # both ranges take the lines of the one with more entries: one launch aggregates them together where it can
        largest = max(plain, key=lambda r: int(p.rowptr[r[1]] - p.rowptr[r[0]]))
        lines = self._lines.get(largest)
        if lines is None:
            lines, _ = _or_none(B.adaqp_spmm_pieces_rule, p.rowptr, p.col, *largest, n_cols, self.dim, self.backward, segments=False) or (0, 0)
        if lines == 0:
            return

        def pieces(begin, end):
            return B.DevicePieces(_or_none(B.adaqp_plan_spmm_pieces, p.rowptr[begin: end + 1], None, self.dim, lines), self.device, begin)
        if (ob, oe) in plain:
            self.pieces_overlap = pieces(ob, oe)
        if (db, de) in plain:
            self.pieces_dependent = pieces(db, de)
        if len(plain) == 2 and oe == db:
            self.pieces_both = pieces(ob, de)

    def _rows_tensor(self):
        """rowptr, whose rows the pieces were planned for, and how often it was written to.  Writes that torch does not count, and those
        that replays and descriptors meet that were taken before, are followed as well, by the kernel and slowly."""
        return self.rowptr, None if self.rowptr.is_inference() else self.rowptr._version

    def _pieces_bytes(self, pieces) -> int:
        return B.adaqp_spmm_pieces_workspace_bytes(pieces.c.n_partials, self.dim)

    def _order_copies(self) -> None:
        """What was just planned is used on the step's streams."""
        for st in (self.stream_msg, self.stream_agg):
            if self._copies():
                st.wait_stream(torch.cuda.current_stream(self.device))

    def _ranges_to_tile(self, tiled: Optional[bool], *ranges):
        """Which of the row ranges of a step are tiled."""
        p, n_cols = self.p, self.p.feat.shape[0]
        if not tiled and n_cols * self.feat.stride(0) * 4 < B.SPMM_SEGMENTS_MOST_BYTES:
            # (a range whose rows do not list ascending, distinct columns has a gain of -infinity and stays as it is)
            rules = [B.adaqp_spmm_pieces_rule(p.rowptr, p.col, b, e, n_cols, self.dim, self.backward) if e > b else (0, -np.inf)
                     for b, e in ranges]
            self._lines = {r: lines for r, (lines, _) in zip(ranges, rules)}
            gains = [gain for _, gain in rules]
            pays = sum(g for g in gains if g > -np.inf) > 0
            return tuple(pays and g > -np.inf for g in gains)
        return tuple(e > b and (tiled or B.adaqp_spmm_tiled_pays(e - b, int(p.rowptr[e] - p.rowptr[b]))) for b, e in ranges)

    def _plan_long_rows(self, begin, end, panels, min_row, piece_cols):
        """Tile table, chunk width, panels or blocks and segments of a row range, and the bytes of workspace these take: partial
        sums of the segments (or of the tiled kernel), then the piece sums of the matrix-core kernel (they may run together)."""
        p, dim, n_cols = self.p, self.dim, self.p.feat.shape[0]
        bounds, off = B.adaqp_plan_spmm_tiles(p.rowptr, p.col, begin, end, n_cols)
        with_panels, with_blocks = B.DevicePanels(None), B.DeviceBlocks(None)
        if panels:
            with_panels = B.DevicePanels(B.adaqp_plan_spmm_panels(p.rowptr, p.col, p.val, begin, end, n_cols, bounds, off, min_row,
                                                                  piece_cols), self.device)
        elif panels is None:
            with_blocks = B.DeviceBlocks(B.adaqp_plan_spmm_blocks(
                p.rowptr, p.col, begin, end, n_cols, dim, B.adaqp_spmm_blocks_min_row(int(bounds[-1])), off,
                only_if_pays_for_ld=self.feat.stride(0), if_slower=bool(self._tiles_asked_for),
                beside=not self.backward), self.device)
            if with_blocks:
                B.adaqp_fill_spmm_blocks(with_blocks, begin, end, self.rowptr, self.col, self.val)
                with_blocks.tensors["copied"] = self.val[int(p.rowptr[begin]): int(p.rowptr[end])].clone()
        segments = B.DeviceSegments(None)
        if n_cols * self.feat.stride(0) * 4 < B.SPMM_SEGMENTS_MOST_BYTES:
            entries = B.adaqp_plan_spmm_segments(p.rowptr, begin, end, bounds, off)
            planned = entries and _or_none(B.adaqp_plan_spmm_pieces, entries["ptr"], entries["of_row"], dim, B.adaqp_spmm_segments_lines(bounds))
            if planned:
                entries["pieces"] = planned
            segments = B.DeviceSegments(entries, self.device)
        if segments:
            B.adaqp_fill_spmm_segments(segments, self.col, self.val)
        need = (B.adaqp_spmm_segments_workspace_bytes(segments, dim) if segments else B.adaqp_spmm_tiled_workspace_bytes(end - begin, dim)) \
            + B.adaqp_spmm_panels_workspace_bytes(with_panels.n_per_tile, dim) \
            + B.adaqp_spmm_blocks_workspace_bytes(with_blocks, dim)
        return (torch.from_numpy(off).to(self.device), B.adaqp_spmm_tiled_chunk_cols(bounds, dim), with_panels, with_blocks,
                segments, need)

    def _plan_dependent(self, panels, min_row, piece_cols) -> int:
        """Tiles the dependent rows; the bytes of workspace that takes."""
        (self.tile_off_dependent, self.tile_chunk_dependent, self.panels_dependent, self.blocks_dependent,
         self.segments_dependent, need) = self._plan_long_rows(*self.p.dependent_rows, panels, min_row, piece_cols)
        return need

    def _copies(self):
        """(blocks, segments, row range) of the ranges that have them."""
        return [c for c in ((self.blocks_overlap, self.segments_overlap, self.p.overlap_rows),
                            (self.blocks_dependent, self.segments_dependent, self.p.dependent_rows)) if c[0] or c[1]]

    def _coefficients(self):
        """val and how often it was written to (None: a tensor that a caller made in inference mode, which does not count that)."""
        return self.val, None if self.val.is_inference() else self.val._version

    def refresh_coefficients(self) -> None:
        """Blocks and segments keep val a second time.  Queues a copy of what has changed in val on stream_msg, which every step
        starts from.  run() and desc() call it when val was written to or replaced, and in every capture, whose replays
        follow val then.  A caller does after writes that torch does not count (through val.data or from a kernel of its own)
        and with a descriptor kept across writes.  Where nothing has changed it costs a read of val and the copies (28 M
        entries 0.11 to 0.12 ms, all of them changed 0.16 to 1.2)."""
        for blocks, segments, (begin, end) in self._copies():
            if blocks:
                B.adaqp_update_spmm_blocks(blocks, begin, end, self.rowptr, self.col, self.val, blocks.tensors["copied"],
                                           self.stream_msg)
            if segments:
                B.adaqp_update_spmm_segments(segments, self.val, self.stream_msg)

    def _follow_coefficients(self) -> None:
        if not self._copies():
            return
        # in a capture whatever val is now: what the replays copy must not hang on when it was last written to
        captured = _capturing(self.stream_msg)
        tensor, version = self._coefficients()
        if captured:
            if not any(kept() is tensor for kept in self._captured):
                self._captured.append(weakref.ref(tensor))
            self.refresh_coefficients()
            return                                  # not made yet
        replays_of_others = any(kept() is not tensor for kept in self._captured)    # may have been copied since
        if tensor is self._copied[0] and version is not None and version == self._copied[1] and not replays_of_others:
            return
        self.refresh_coefficients()
        self._copied = tensor, version

    def set_fused_receive(self, on: bool) -> None:
        """Forward only.  On: received rows are not de-quantised into feat; the dependent aggregation reads
        them from the receive buffer.  Off, in a step that was made with it on: plans the tiles of the dependent rows."""
        self.fused_receive = bool(on) and not self.backward and self.plan.halo_idx_host is not None
        if self.fused_receive and self.slot_of_row is None:
            # scratch of each step; before the upload, which waits for whatever its memory was used for
            self.packed_row = torch.empty((self.p.feat.shape[0], 2), dtype=torch.int32, device=self.device)
            self.slot_of_row = torch.from_numpy(
                B.adaqp_plan_slot_of_row(self.p.feat.shape[0], self.plan.halo_idx_host)).to(self.device)
        if not self.fused_receive and self._unplanned_dependent is not None:
            tiled, *how = self._unplanned_dependent
            self._unplanned_dependent = None
            if self._ranges_to_tile(tiled, self.p.dependent_rows)[0]:
                need = self._plan_dependent(*how)
                if need > self.ws_dependent.numel():                # descriptors that were taken before name the former one
                    self._former_workspace = self.ws_dependent
                    self.ws_dependent = torch.empty(need, dtype=torch.uint8, device=self.device)
                self._order_copies()

    def desc(self, schedule: int) -> B.LayerDesc:
        self._follow_coefficients()
        p, pl = self.p, self.plan
        d = B.LayerDesc()
        d.direction = B.BACKWARD if self.backward else B.FORWARD
        d.schedule = schedule
        d.rowptr_dev, d.col_dev, d.val_dev = self.rowptr.data_ptr(), self.col.data_ptr(), self.val.data_ptr()
        d.nnz = p.nnz
        d.overlap_begin, d.overlap_end = p.overlap_rows
        d.dependent_begin, d.dependent_end = p.dependent_rows
        d.overlap_nnz, d.dependent_nnz = self.overlap_nnz, self.dependent_nnz
        d.feat_dev, d.n_feat_rows, d.ld, d.dim = self.feat.data_ptr(), self.feat.shape[0], self.feat.stride(0), self.dim
        d.out_dev, d.ldo = self.out.data_ptr(), self.out.stride(0)
        d.send_idx_dev, d.bits_dev = pl.send_idx.data_ptr(), pl.bits.data_ptr()
        d.row_offset_dev = pl.row_offset.data_ptr()
        d.halo_idx_dev = None if pl.halo_idx is None else pl.halo_idx.data_ptr()
        d.recv_order_dev = pl.recv_order.data_ptr() if (self.use_recv_order and pl.recv_order is not None
                                                        and not self.backward) else None
        d.slot_of_row_dev = self.slot_of_row.data_ptr() if self.fused_receive else None
        # (filled for every row of feat: not where a caller has put a taller matrix in its place)
        tables = min(self.packed_row.shape[0], self.slot_of_row.shape[0]) if self.fused_receive else 0
        d.packed_row_dev = self.packed_row.data_ptr() if tables >= self.feat.shape[0] > 0 else None
        d.tile_off_overlap_dev = None if self.tile_off_overlap is None else self.tile_off_overlap.data_ptr()
        d.tile_chunk_overlap, d.tile_chunk_dependent = self.tile_chunk_overlap, self.tile_chunk_dependent
        d.tile_off_dependent_dev = None if (self.tile_off_dependent is None or self.fused_receive) \
            else self.tile_off_dependent.data_ptr()
        if d.tile_off_overlap_dev:
            d.panels_overlap, d.blocks_overlap = self.panels_overlap.c, self.blocks_overlap.c
            d.segments_overlap = self.segments_overlap.c
        if d.tile_off_dependent_dev:
            d.panels_dependent, d.blocks_dependent = self.panels_dependent.c, self.blocks_dependent.c
            d.segments_dependent = self.segments_dependent.c
        if self.backward and self.backward_receive and pl.seg_order is not None:
            d.recv_seg_order_dev, d.recv_seg_ptr_dev = pl.seg_order.data_ptr(), pl.seg_ptr.data_ptr()
            d.n_recv_seg = pl.seg_ptr.shape[0] - 1
        d.n_send, d.seed = pl.n, self.seed
        d.packed_dev, d.params_dev = self.packed.data_ptr(), self.params.data_ptr()
        if self.alpha_sq is not None:
            d.alpha_sq_dev, d.beta_dev = self.alpha_sq.data_ptr(), self.beta.data_ptr()
        d.recv_packed_dev, d.recv_params_dev = self.recv_packed.data_ptr(), self.recv_params.data_ptr()
        d.packed_bytes = pl.packed_bytes
        d.workspace_overlap_dev, d.workspace_overlap_bytes = self.ws_overlap.data_ptr(), self.ws_overlap.numel()
        d.workspace_dependent_dev, d.workspace_dependent_bytes = self.ws_dependent.data_ptr(), self.ws_dependent.numel()
        d.stream_msg = self.stream_msg.cuda_stream
        d.stream_agg = self.stream_agg.cuda_stream
        d.event_fork, d.event_join = self.event_fork.handle, self.event_join.handle
        if self._rows_tensor()[0] is self._planned_rows[0] and self._rows_tensor()[1] == self._planned_rows[1]:     # else: cut on the device
            d.pieces_overlap, d.pieces_dependent, d.pieces_both = self.pieces_overlap.c, self.pieces_dependent.c, self.pieces_both.c
        return d

    def default_schedule(self) -> int:
        """CHAIN where a second stream has nothing to hide or to pair, else ISOLATED."""
        dependent = self.tile_off_dependent is not None and not self.fused_receive
        tiled, both = self.tile_off_overlap is not None or dependent, self.tile_off_overlap is not None and dependent
        # two tiled aggregations wait for each other, so that a second stream only hides the messages (58 000 rows, 28 M entries,
        # 256 columns: 1.59 ms in a row, 1.64 on two streams), but pairs with what matrix-core kernels leave of the GPU
        matrix = self.panels_overlap or self.panels_dependent or self.blocks_overlap or self.blocks_dependent
        alone = not tiled or (both and not matrix)
        return B.CHAIN if alone and self.plan.packed_bytes <= CHAIN_BYTES else B.ISOLATED

    def run(self, schedule: Optional[int] = None) -> None:
        """Enqueues one layer step; synchronise stream_msg to wait for it.  Without a schedule the step takes the one of
        default_schedule(): work that a caller queues on stream_agg itself is ordered with such a step through stream_msg
        only.  A schedule that is given is kept."""
        B.adaqp_layer_step(self.desc(self.default_schedule() if schedule is None else schedule))

    def synchronize(self) -> None:
        self.stream_msg.synchronize()
        self.stream_agg.synchronize()
