"""Thin ctypes binding of libadaqp.so (include/adaqp.h).  Argument marshalling only.

Every function has the name of the C entry point it calls.  Tensors are torch tensors that already live
where the C function expects them (device tensors for *_dev arguments, numpy arrays for the host-only
layout call); torch supplies device memory and streams and nothing else.  There is no fallback: if the
library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

import numpy as np
import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libadaqp.so")

OK, EINVAL, EBITS, ESIZE, EHIP = 0, -1, -2, -3, -4
SERIAL, ISOLATED, FREE, CHAIN = 0, 1, 2, 3
FORWARD, BACKWARD = 0, 1

_i64, _i32, _u64, _vp = ctypes.c_int64, ctypes.c_int32, ctypes.c_uint64, ctypes.c_void_p


class AdaqpError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        L = lib()
        msg = L.adaqp_strerror(status).decode()
        if status == EHIP:
            msg += ": " + L.adaqp_last_hip_error().decode()
        super().__init__(f"{where}: {msg} ({status})")


class SpmmPanels(ctypes.Structure):
    """Mirror of struct adaqp_spmm_panels."""
    _fields_ = [
        ("n_panels", _i32), ("n_per_tile", _i32), ("n_groups", _i64), ("n_panel_pieces", _i64),
        ("panel_rows_dev", _vp), ("pcol_dev", _vp), ("palpha_dev", _vp), ("piece_dev", _vp),
        ("panel_piece_ptr_dev", _vp), ("panel_piece_dev", _vp),
    ]


class SpmmBlocks(ctypes.Structure):
    """Mirror of struct adaqp_spmm_blocks."""
    _fields_ = [
        ("n_blocks", _i32), ("n_pieces", _i32), ("n_steps", _i64), ("col_begin", _i32), ("piece_width", _i32),
        ("rows_dev", _vp), ("step_ptr_dev", _vp), ("cols_dev", _vp), ("table_dev", _vp),
    ]


class SpmmPieces(ctypes.Structure):
    """Mirror of struct adaqp_spmm_pieces."""
    _fields_ = [
        ("n_pieces", _i64), ("n_partials", _i64), ("n_sums", _i64), ("n_seg", _i64), ("row_begin", _i64),
        ("lines_per_slice", _i32), ("waves", _i32), ("entries", _i32), ("reserved", _i32),
        ("pieces_dev", _vp), ("dest_dev", _vp), ("sum_row_dev", _vp), ("sum_ptr_dev", _vp),
    ]


class SpmmSegments(ctypes.Structure):
    """Mirror of struct adaqp_spmm_segments."""
    _fields_ = [
        ("n_seg", _i64), ("n_entries", _i64), ("n_rows", _i64), ("ptr_dev", _vp), ("src_dev", _vp), ("of_row_dev", _vp),
        ("col_dev", _vp), ("val_dev", _vp), ("pieces", SpmmPieces),
    ]


class LayerDesc(ctypes.Structure):
    """Mirror of struct adaqp_layer_desc."""
    _fields_ = [
        ("direction", _i32), ("schedule", _i32),
        ("rowptr_dev", _vp), ("col_dev", _vp), ("val_dev", _vp), ("nnz", _i64),
        ("overlap_begin", _i64), ("overlap_end", _i64), ("overlap_nnz", _i64),
        ("dependent_begin", _i64), ("dependent_end", _i64), ("dependent_nnz", _i64),
        ("feat_dev", _vp), ("n_feat_rows", _i64), ("ld", _i64), ("dim", _i32),
        ("out_dev", _vp), ("ldo", _i64),
        ("send_idx_dev", _vp), ("bits_dev", _vp), ("row_offset_dev", _vp), ("halo_idx_dev", _vp),
        ("recv_order_dev", _vp),
        ("slot_of_row_dev", _vp),
        ("tile_off_overlap_dev", _vp), ("tile_off_dependent_dev", _vp),
        ("tile_chunk_overlap", _i32), ("tile_chunk_dependent", _i32),
        ("panels_overlap", SpmmPanels), ("panels_dependent", SpmmPanels),
        ("blocks_overlap", SpmmBlocks), ("blocks_dependent", SpmmBlocks),
        ("segments_overlap", SpmmSegments), ("segments_dependent", SpmmSegments),
        ("recv_seg_order_dev", _vp), ("recv_seg_ptr_dev", _vp), ("n_recv_seg", _i64),
        ("n_send", _i64), ("seed", _u64),
        ("packed_dev", _vp), ("params_dev", _vp), ("alpha_sq_dev", _vp), ("beta_dev", _vp),
        ("recv_packed_dev", _vp), ("recv_params_dev", _vp),
        ("packed_bytes", _i64),
        ("workspace_overlap_dev", _vp), ("workspace_overlap_bytes", _i64),
        ("workspace_dependent_dev", _vp), ("workspace_dependent_bytes", _i64),
        ("stream_msg", _vp), ("stream_agg", _vp), ("event_fork", _vp), ("event_join", _vp),
        ("packed_row_dev", _vp),
        ("pieces_overlap", SpmmPieces), ("pieces_dependent", SpmmPieces), ("pieces_both", SpmmPieces),
    ]


_lib: Optional[ctypes.CDLL] = None

_SIGNATURES = {
    "adaqp_strerror": (ctypes.c_char_p, [ctypes.c_int]),
    "adaqp_last_hip_error": (ctypes.c_char_p, []),
    "adaqp_version": (ctypes.c_int, []),
    "adaqp_row_stride": (_i64, [_i32, _i32]),
    "adaqp_plan_layout": (ctypes.c_int, [_i64, _i32, _vp, _vp, _i32, _vp, _vp, _vp]),
    "adaqp_quantize_pack": (ctypes.c_int, [_vp, _i64, _i64, _i32, _vp, _vp, _vp, _i64, _u64, _vp, _i64, _vp, _vp]),
    "adaqp_quantize_pack_trace": (ctypes.c_int, [_vp, _i64, _i64, _i32, _vp, _vp, _vp, _i64, _u64, _vp, _i64, _vp,
                                                 _vp, _vp, _vp]),
    "adaqp_plan_send": (ctypes.c_int, [_i64, _i32, _vp, _vp, _i32] + [_vp] * 9),
    "adaqp_plan_recv_order": (ctypes.c_int, [_i64, _vp, _vp]),
    "adaqp_unpack_dequant": (ctypes.c_int, [_vp, _i64, _vp, _vp, _vp, _vp, _vp, _i64, _i32, _vp, _i64, _i64, _vp]),
    "adaqp_plan_recv_segments": (ctypes.c_int, [_i64, _vp, _vp, _vp, ctypes.POINTER(_i64)]),
    "adaqp_unpack_dequant_add": (ctypes.c_int, [_vp, _i64, _vp, _vp, _vp, _vp, _i64, _vp, _vp, _i64, _i32,
                                                _vp, _i64, _i64, _vp]),
    "adaqp_spmm_workspace_bytes": (ctypes.c_int, [_i64, _i64, _i32, ctypes.POINTER(_i64)]),
    "adaqp_spmm_csr": (ctypes.c_int, [_vp, _vp, _vp, _i64, _i64, _i64, _i64, _vp, _i64, _i64, _i32,
                                      _vp, _i64, _vp, _i64, _vp]),
    "adaqp_spmm_csr_noalloc": (ctypes.c_int, [_vp, _vp, _vp, _i64, _i64, _i64, _i64, _vp, _i64, _i64, _i32,
                                              _vp, _i64, _vp]),
    "adaqp_plan_spmm_tiles": (ctypes.c_int, [_vp, _vp, _i64, _i64, _i64, _vp, _vp]),
    "adaqp_spmm_tiled_workspace_bytes": (ctypes.c_int, [_i64, _i32, _vp]),
    "adaqp_spmm_tiled_pays": (_i32, [_i64, _i64]),
    "adaqp_spmm_tiled_chunk_cols": (_i32, [_vp, _i32]),
    "adaqp_spmm_csr_tiled": (ctypes.c_int, [_vp, _vp, _vp, _i64, _i64, _i64, _vp, _i64, _i64, _i32, _vp, _i64,
                                            _vp, _i32, _vp, _i64, _vp]),
    "adaqp_plan_spmm_panels": (ctypes.c_int, [_vp, _vp, _vp, _i64, _i64, _i64, _vp, _i32, _i32, _vp, _vp, _vp, _vp,
                                              _vp, _vp, _vp, _vp]),
    "adaqp_spmm_panels_workspace_bytes": (ctypes.c_int, [_i32, _i32, _vp]),
    "adaqp_spmm_panels_pay": (_i32, [_i64, _i32]),
    "adaqp_spmm_segments_gain": (ctypes.c_int, [_vp, _vp, _i64, _i64, _i64, _i32, _i32, _vp]),
    "adaqp_plan_spmm_segments": (ctypes.c_int, [_vp, _i64, _i64, _vp, _vp, _vp, _vp, _vp, _vp]),
    "adaqp_plan_packed_rows": (ctypes.c_int, [_i64, _i64, _vp, _vp, _vp, _i32, _i64, _vp]),
    "adaqp_spmm_pieces_rule": (ctypes.c_int, [_vp, _vp, _i64, _i64, _i64, _i32, _i32, _vp, _vp]),
    "adaqp_spmm_segments_lines": (_i32, [_vp]),
    "adaqp_plan_spmm_pieces": (ctypes.c_int, [_vp, _i64, _vp, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _vp]),
    "adaqp_spmm_pieces_workspace_bytes": (ctypes.c_int, [_i64, _i32, _vp]),
    "adaqp_fill_spmm_segments": (ctypes.c_int, [ctypes.POINTER(SpmmSegments), _vp, _vp, _i64, _vp]),
    "adaqp_update_spmm_segments": (ctypes.c_int, [ctypes.POINTER(SpmmSegments), _vp, _i64, _vp]),
    "adaqp_spmm_segments_workspace_bytes": (ctypes.c_int, [_i64, _i64, _i32, _vp]),
    "adaqp_spmm_csr_segments": (ctypes.c_int, [ctypes.POINTER(SpmmSegments), _vp, _i64, _i64, _i32, _vp, _i64, _vp, _i64, _vp]),
    "adaqp_plan_spmm_blocks": (ctypes.c_int, [_vp, _vp, _i64, _i64, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _vp]),
    "adaqp_spmm_blocks_min_row": (_i32, [_i64]),
    "adaqp_spmm_blocks_pay": (_i32, [_i64, _i64, _i64]),
    "adaqp_spmm_blocks_save": (_i32, [_i64, _i64, _i32, _i32]),
    "adaqp_spmm_blocks_most_steps": (_i64, [_i64]),
    "adaqp_spmm_blocks_table_floats": (_i64, [_i64]),
    "adaqp_fill_spmm_blocks": (ctypes.c_int, [ctypes.POINTER(SpmmBlocks), _i64, _i64, _vp, _vp, _vp, _i64, _vp]),
    "adaqp_update_spmm_blocks": (ctypes.c_int, [ctypes.POINTER(SpmmBlocks), _i64, _i64, _vp, _vp, _vp, _i64, _vp, _vp]),
    "adaqp_spmm_blocks_workspace_bytes": (ctypes.c_int, [_i32, _i32, _i32, _vp]),
    "adaqp_spmm_csr_blocks": (ctypes.c_int, [ctypes.POINTER(SpmmBlocks), _i64, _i64, _vp, _i64, _i64, _i32, _vp, _i64, _vp, _i64,
                                             _vp]),
    "adaqp_spmm_csr_panels": (ctypes.c_int, [ctypes.POINTER(SpmmPanels), _i64, _i64, _vp, _i64, _i64, _i32, _vp,
                                             _i64, _vp, _i64, _vp]),
    "adaqp_assign_bits": (ctypes.c_int, [_i64, _vp, _vp, _i32, _i32, _i32, ctypes.c_double, _vp, _vp, _vp, _vp]),
    "adaqp_plan_slot_of_row": (ctypes.c_int, [_i64, _i64, _vp, _vp]),
    "adaqp_spmm_csr_packed": (ctypes.c_int, [_vp, _vp, _vp, _i64, _i64, _i64, _i64, _vp, _i64, _i64, _i32,
                                             _vp, _i64, _vp, _vp, _i64, _vp, _vp, _vp, _i64, _vp, _i64, _vp]),
    "adaqp_layer_step": (ctypes.c_int, [ctypes.POINTER(LayerDesc)]),
    "adaqp_probe_quantize_pack": (ctypes.c_int, [_vp, _i64, _i64, _i32, _vp, _vp, _vp, _i64, _vp, _i64, _vp, _vp]),
    "adaqp_probe_unpack_dequant_add": (ctypes.c_int, [_vp, _i64, _vp, _vp, _vp, _vp, _i64, _vp, _vp, _i64, _i32,
                                                _vp, _i64, _i64, _vp]),
    "adaqp_probe_stream": (ctypes.c_int, [_vp, _vp, _i64, _i32, _vp]),
    "adaqp_probe_xcd_of_workgroup": (ctypes.c_int, [_vp, _i32, _vp]),
    "adaqp_layer_desc_bytes": (_i64, []),
}
EXPORTS = tuple(_SIGNATURES)


def lib() -> ctypes.CDLL:
    """Loads the in-tree library; raises if it has not been built (python -m paper_2306_01381_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_2306_01381_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        if int(L.adaqp_layer_desc_bytes()) != ctypes.sizeof(LayerDesc):
            raise ImportError(f"LayerDesc ({ctypes.sizeof(LayerDesc)} bytes) does not mirror adaqp_layer_desc "
                              f"({int(L.adaqp_layer_desc_bytes())} bytes) of {LIB_PATH}: rebuild the library")
        _lib = L
    return _lib


def _check(status: int, where: str) -> None:
    if status != OK:
        raise AdaqpError(status, where)


def _dev(t: Optional[torch.Tensor], dtype: torch.dtype, name: str) -> Optional[int]:
    if t is None:
        return None
    if not t.is_cuda:
        raise TypeError(f"{name} must be a device tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise TypeError(f"{name} must be contiguous")
    return t.data_ptr()


def _stream(stream: Optional[torch.cuda.Stream]) -> Optional[int]:
    s = torch.cuda.current_stream() if stream is None else stream
    return s.cuda_stream or None


def _matrix(t: torch.Tensor, name: str) -> Tuple[int, int, int]:
    """(pointer, rows, leading dimension) of a 2-D fp32 device tensor whose rows are contiguous."""
    if not t.is_cuda or t.dtype != torch.float32 or t.dim() != 2 or t.stride(1) != 1:
        raise TypeError(f"{name} must be a 2-D fp32 device tensor with unit column stride")
    return t.data_ptr(), t.shape[0], t.stride(0) if t.shape[0] > 1 else max(t.stride(0), t.shape[1])


def adaqp_version() -> int:
    return lib().adaqp_version()


def adaqp_row_stride(dim: int, bits: int) -> int:
    return int(lib().adaqp_row_stride(dim, bits))


def adaqp_plan_layout(dim: int, bits_host: np.ndarray, peer_of_slot_host: np.ndarray, n_peers: int):
    """Host-only.  Returns (perm, row_offset, peer_byte_ptr) as int64 numpy arrays."""
    bits = np.ascontiguousarray(bits_host, dtype=np.uint8)
    peer = np.ascontiguousarray(peer_of_slot_host, dtype=np.int32)
    n = bits.shape[0]
    if peer.shape[0] != n:
        raise ValueError("bits and peer_of_slot differ in length")
    perm = np.zeros(n, dtype=np.int64)
    off = np.zeros(n, dtype=np.int64)
    pbp = np.zeros(max(n_peers, 0) + 1, dtype=np.int64)
    _check(lib().adaqp_plan_layout(n, dim, bits.ctypes.data, peer.ctypes.data, n_peers,
                                   perm.ctypes.data, off.ctypes.data, pbp.ctypes.data), "adaqp_plan_layout")
    return perm, off, pbp


def adaqp_plan_send(dim: int, bits_host: np.ndarray, peer_of_slot_host: np.ndarray, n_peers: int, send_idx_host: np.ndarray,
                    halo_idx_host: Optional[np.ndarray]) -> dict:
    """Host-only.  adaqp_plan_layout's perm, row_offset and peer_byte_ptr, and the per-slot arrays in sorted order: send_idx, bits and (with
    halo_idx) halo_idx, recv_order.  `blob` (uint8) holds what the device needs, every array but perm and peer_byte_ptr, each at a multiple of
    256 bytes named in `at`: one upload."""
    bits = np.ascontiguousarray(bits_host, dtype=np.uint8)
    peer = np.ascontiguousarray(peer_of_slot_host, dtype=np.int32)
    n = bits.shape[0]
    if peer.shape[0] != n:
        raise ValueError("bits and peer_of_slot differ in length")
    arrays = [("row_offset", np.int64), ("send_idx", np.int32)] + ([("halo_idx", np.int32), ("recv_order", np.int32)] if halo_idx_host is not None else []) \
        + [("bits", np.uint8)]
    send = np.ascontiguousarray(send_idx_host, dtype=np.int32)
    halo = None if halo_idx_host is None else np.ascontiguousarray(halo_idx_host, dtype=np.int32)
    if send.shape[0] < n or (halo is not None and halo.shape[0] < n):
        raise IndexError("send_idx or halo_idx has fewer entries than slots")
    at, total = {}, 0
    for name, dtype in arrays:
        at[name] = (total, n * np.dtype(dtype).itemsize, dtype)
        total += -(-at[name][1] // 256) * 256
    plan = {"perm": np.empty(n, dtype=np.int64), "peer_byte_ptr": np.zeros(max(n_peers, 0) + 1, dtype=np.int64),
            "blob": np.empty(total, dtype=np.uint8), "at": at}
    for name, (begin, size, dtype) in at.items():
        plan[name] = plan["blob"][begin:begin + size].view(dtype)

    def ptr(name):
        return plan[name].ctypes.data if name in plan else None
    _check(lib().adaqp_plan_send(n, dim, bits.ctypes.data, peer.ctypes.data, n_peers, send.ctypes.data, None if halo is None else halo.ctypes.data,
                                 ptr("perm"), ptr("row_offset"), ptr("peer_byte_ptr"), ptr("send_idx"), ptr("bits"), ptr("halo_idx"),
                                 ptr("recv_order")), "adaqp_plan_send")
    return plan


def adaqp_quantize_pack(feat: torch.Tensor, dim: int, send_idx: torch.Tensor, bits: torch.Tensor,
                        row_offset: torch.Tensor, seed: int, packed: torch.Tensor, params: torch.Tensor,
                        stream: Optional[torch.cuda.Stream] = None) -> None:
    fp, n_rows, ld = _matrix(feat, "feat")
    n = send_idx.shape[0]
    _check(lib().adaqp_quantize_pack(fp, n_rows, ld, dim, _dev(send_idx, torch.int32, "send_idx"),
                                     _dev(bits, torch.uint8, "bits"), _dev(row_offset, torch.int64, "row_offset"),
                                     n, seed & (2**64 - 1), _dev(packed, torch.uint8, "packed"), packed.numel(),
                                     _dev(params, torch.float32, "params"), _stream(stream)),
           "adaqp_quantize_pack")


def adaqp_quantize_pack_trace(feat: torch.Tensor, dim: int, send_idx: torch.Tensor, bits: torch.Tensor,
                              row_offset: torch.Tensor, seed: int, packed: torch.Tensor, params: torch.Tensor,
                              alpha_sq: torch.Tensor, beta: torch.Tensor,
                              stream: Optional[torch.cuda.Stream] = None) -> None:
    fp, n_rows, ld = _matrix(feat, "feat")
    n = send_idx.shape[0]
    _check(lib().adaqp_quantize_pack_trace(fp, n_rows, ld, dim, _dev(send_idx, torch.int32, "send_idx"),
                                           _dev(bits, torch.uint8, "bits"),
                                           _dev(row_offset, torch.int64, "row_offset"), n, seed & (2**64 - 1),
                                           _dev(packed, torch.uint8, "packed"), packed.numel(),
                                           _dev(params, torch.float32, "params"),
                                           _dev(alpha_sq, torch.float32, "alpha_sq"),
                                           _dev(beta, torch.float32, "beta"), _stream(stream)),
           "adaqp_quantize_pack_trace")


def adaqp_plan_recv_order(halo_idx_host: np.ndarray) -> np.ndarray:
    """Host-only.  Returns the int32 visiting order of the receive slots (ascending destination rows)."""
    halo = np.ascontiguousarray(halo_idx_host, dtype=np.int32)
    order = np.zeros(halo.shape[0], dtype=np.int32)
    _check(lib().adaqp_plan_recv_order(halo.shape[0], halo.ctypes.data, order.ctypes.data), "adaqp_plan_recv_order")
    return order


def adaqp_unpack_dequant(packed: torch.Tensor, params: torch.Tensor, bits: torch.Tensor,
                         row_offset: torch.Tensor, halo_idx: torch.Tensor, dim: int, feat: torch.Tensor,
                         order: Optional[torch.Tensor] = None,
                         stream: Optional[torch.cuda.Stream] = None) -> None:
    fp, n_rows, ld = _matrix(feat, "feat")
    n = halo_idx.shape[0]
    _check(lib().adaqp_unpack_dequant(_dev(packed, torch.uint8, "packed"), packed.numel(),
                                      _dev(params, torch.float32, "params"), _dev(bits, torch.uint8, "bits"),
                                      _dev(row_offset, torch.int64, "row_offset"),
                                      _dev(halo_idx, torch.int32, "halo_idx"), _dev(order, torch.int32, "order"),
                                      n, dim, fp, n_rows, ld,
                                      _stream(stream)),
           "adaqp_unpack_dequant")


def adaqp_plan_recv_segments(dst_idx_host: np.ndarray):
    """Host-only.  Returns (order int32[n], seg_ptr int64[n_seg + 1])."""
    dst = np.ascontiguousarray(dst_idx_host, dtype=np.int32)
    n = dst.shape[0]
    order = np.zeros(n, dtype=np.int32)
    seg_ptr = np.zeros(n + 1, dtype=np.int64)
    n_seg = _i64(0)
    _check(lib().adaqp_plan_recv_segments(n, dst.ctypes.data, order.ctypes.data, seg_ptr.ctypes.data,
                                          ctypes.byref(n_seg)), "adaqp_plan_recv_segments")
    return order, seg_ptr[: n_seg.value + 1].copy()


def adaqp_unpack_dequant_add(packed: torch.Tensor, params: torch.Tensor, bits: torch.Tensor,
                             row_offset: torch.Tensor, dst_idx: torch.Tensor, seg_order: torch.Tensor,
                             seg_ptr: torch.Tensor, dim: int, grad: torch.Tensor,
                             stream: Optional[torch.cuda.Stream] = None) -> None:
    gp, n_rows, ld = _matrix(grad, "grad")
    _check(lib().adaqp_unpack_dequant_add(_dev(packed, torch.uint8, "packed"), packed.numel(),
                                          _dev(params, torch.float32, "params"), _dev(bits, torch.uint8, "bits"),
                                          _dev(row_offset, torch.int64, "row_offset"),
                                          _dev(dst_idx, torch.int32, "dst_idx"), dst_idx.shape[0],
                                          _dev(seg_order, torch.int32, "seg_order"),
                                          _dev(seg_ptr, torch.int64, "seg_ptr"), seg_ptr.shape[0] - 1,
                                          dim, gp, n_rows, ld, _stream(stream)),
           "adaqp_unpack_dequant_add")


def adaqp_spmm_workspace_bytes(n_rows: int, nnz: int, dim: int) -> int:
    out = _i64(0)
    _check(lib().adaqp_spmm_workspace_bytes(n_rows, nnz, dim, ctypes.byref(out)), "adaqp_spmm_workspace_bytes")
    return int(out.value)


def adaqp_spmm_csr(rowptr: torch.Tensor, col: torch.Tensor, val: torch.Tensor, row_begin: int, row_end: int,
                   H: torch.Tensor, dim: int, out: torch.Tensor, workspace: torch.Tensor,
                   nnz_range: int = -1, stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr(_dev(rowptr, torch.int64, "rowptr"), _dev(col, torch.int32, "col"),
                                _dev(val, torch.float32, "val"), col.numel(), row_begin, row_end, nnz_range,
                                hp, n_cols, ldh, dim, op, ldo, _dev(workspace, torch.uint8, "workspace"),
                                workspace.numel(), _stream(stream)),
           "adaqp_spmm_csr")


SPMM_NOALLOC_SCRATCH_BYTES = 64 << 20


def adaqp_spmm_csr_noalloc(rowptr: torch.Tensor, col: torch.Tensor, val: torch.Tensor, row_begin: int, row_end: int,
                           H: torch.Tensor, dim: int, out: torch.Tensor, nnz_range: int = -1,
                           stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr_noalloc(_dev(rowptr, torch.int64, "rowptr"), _dev(col, torch.int32, "col"),
                                        _dev(val, torch.float32, "val"), col.numel(), row_begin, row_end, nnz_range,
                                        hp, n_cols, ldh, dim, op, ldo, _stream(stream)),
           "adaqp_spmm_csr_noalloc")


SPMM_TILES = 8
SPMM_TILED_SHORT_ROW = 64
SPMM_PANEL_ROWS = 32
SPMM_PANEL_MIN_ROW = 6144
SPMM_PANEL_PIECE_COLS = 1024


def adaqp_plan_spmm_tiles(rowptr_host: np.ndarray, col_host: np.ndarray, row_begin: int, row_end: int,
                          n_cols: int) -> Tuple[np.ndarray, np.ndarray]:
    """Host-only.  Returns (col_bounds int32[9], tile_off int32[rows, 9])."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    col = np.ascontiguousarray(col_host, dtype=np.int32)
    bounds = np.zeros(SPMM_TILES + 1, dtype=np.int32)
    off = np.zeros((max(row_end - row_begin, 0), SPMM_TILES + 1), dtype=np.int32)
    _check(lib().adaqp_plan_spmm_tiles(rowptr.ctypes.data, col.ctypes.data, row_begin, row_end, n_cols,
                                       bounds.ctypes.data, off.ctypes.data), "adaqp_plan_spmm_tiles")
    return bounds, off


def adaqp_spmm_tiled_workspace_bytes(n_rows: int, dim: int) -> int:
    out = ctypes.c_int64(0)
    _check(lib().adaqp_spmm_tiled_workspace_bytes(n_rows, dim, ctypes.byref(out)), "adaqp_spmm_tiled_workspace_bytes")
    return int(out.value)


def adaqp_spmm_tiled_pays(n_rows: int, nnz: int) -> bool:
    """Host-only.  True if a row range of this shape is better served by adaqp_spmm_csr_tiled."""
    return bool(lib().adaqp_spmm_tiled_pays(n_rows, nnz))


def adaqp_spmm_tiled_chunk_cols(col_bounds_host: np.ndarray, dim: int) -> int:
    """Host-only.  64 or 128: the feature-chunk width for a plan with these column bounds."""
    b = np.ascontiguousarray(col_bounds_host, dtype=np.int32)
    if b.shape[0] != SPMM_TILES + 1:
        raise ValueError("col_bounds needs SPMM_TILES + 1 entries")
    c = int(lib().adaqp_spmm_tiled_chunk_cols(b.ctypes.data, dim))
    if c == 0:
        raise AdaqpError("adaqp_spmm_tiled_chunk_cols", -1)
    return c


def adaqp_plan_spmm_panels(rowptr_host: np.ndarray, col_host: np.ndarray, val_host: np.ndarray, row_begin: int,
                           row_end: int, n_cols: int, col_bounds_host: np.ndarray,
                           tile_off: Optional[np.ndarray] = None, min_row_len: int = SPMM_PANEL_MIN_ROW,
                           piece_cols: int = SPMM_PANEL_PIECE_COLS, only_if_pays_for_dim: int = 0) -> Optional[dict]:
    """Host-only.  Returns None when no row of the range has min_row_len entries (or, with only_if_pays_for_dim =
    the row width, when adaqp_spmm_panels_pay turns the sized plan down), else a dict of host arrays
    (panel_rows, pcol, palpha, piece, panel_piece_ptr, panel_piece) and sizes (n_rows_taken, n_panels, n_groups,
    n_per_tile, n_panel_pieces).  tile_off (the C-contiguous int32 table of adaqp_plan_spmm_tiles for the same
    range) is changed in place: the rows taken are struck from it."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    col = np.ascontiguousarray(col_host, dtype=np.int32)
    val = np.ascontiguousarray(val_host, dtype=np.float32)
    bounds = np.ascontiguousarray(col_bounds_host, dtype=np.int32)
    if bounds.shape[0] != SPMM_TILES + 1:
        raise ValueError("col_bounds needs SPMM_TILES + 1 entries")
    if tile_off is not None:
        if tile_off.dtype != np.int32 or not tile_off.flags.c_contiguous or \
                tile_off.shape != (max(row_end - row_begin, 0), SPMM_TILES + 1):
            raise ValueError("tile_off must be the C-contiguous int32 table of adaqp_plan_spmm_tiles for this range")
    sizes = np.zeros(5, dtype=np.int64)
    args = (rowptr.ctypes.data, col.ctypes.data, val.ctypes.data, row_begin, row_end, n_cols, bounds.ctypes.data,
            min_row_len, piece_cols, sizes.ctypes.data)
    _check(lib().adaqp_plan_spmm_panels(*args, None, None, None, None, None, None, None), "adaqp_plan_spmm_panels")
    taken, n_panels, n_groups, n_per_tile, n_pieces = (int(x) for x in sizes)
    if taken == 0:
        return None
    if only_if_pays_for_dim > 0 and not adaqp_spmm_panels_pay(n_pieces, only_if_pays_for_dim):
        return None
    plan = {
        "n_rows_taken": taken, "n_panels": n_panels, "n_groups": n_groups, "n_per_tile": n_per_tile,
        "n_panel_pieces": n_pieces,
        "panel_rows": np.empty(n_panels * SPMM_PANEL_ROWS, dtype=np.int32),
        "pcol": np.empty((n_groups, 2, 4), dtype=np.int32),
        "palpha": np.empty((n_groups, 64, 4), dtype=np.float32),
        "piece": np.empty((SPMM_TILES, n_per_tile, 2), dtype=np.int32),
        "panel_piece_ptr": np.empty(n_panels + 1, dtype=np.int32),
        "panel_piece": np.empty(n_pieces, dtype=np.int32),
    }
    _check(lib().adaqp_plan_spmm_panels(*args, None if tile_off is None else tile_off.ctypes.data,
                                        plan["panel_rows"].ctypes.data, plan["pcol"].ctypes.data,
                                        plan["palpha"].ctypes.data, plan["piece"].ctypes.data,
                                        plan["panel_piece_ptr"].ctypes.data, plan["panel_piece"].ctypes.data),
           "adaqp_plan_spmm_panels")
    return plan


class DevicePanels:
    """Device copies of a panel plan plus the struct the C calls take.  Keeps the tensors alive."""

    def __init__(self, plan: Optional[dict], device="cuda"):
        self.c = SpmmPanels()
        self.tensors = {}
        self.n_per_tile = 0
        if plan is None:
            return
        for k in ("panel_rows", "pcol", "palpha", "piece", "panel_piece_ptr", "panel_piece"):
            self.tensors[k] = torch.from_numpy(plan[k]).to(device)
        t = self.tensors
        self.n_per_tile = plan["n_per_tile"]
        self.c = SpmmPanels(plan["n_panels"], plan["n_per_tile"], plan["n_groups"], plan["n_panel_pieces"],
                            t["panel_rows"].data_ptr(), t["pcol"].data_ptr(), t["palpha"].data_ptr(),
                            t["piece"].data_ptr(), t["panel_piece_ptr"].data_ptr(), t["panel_piece"].data_ptr())

    def __bool__(self) -> bool:
        return self.c.n_panels > 0


def adaqp_spmm_panels_pay(n_panel_pieces: int, dim: int) -> bool:
    """Host-only.  True if a panel plan of that many pieces is worth launching (it fills enough of the GPU)."""
    return bool(lib().adaqp_spmm_panels_pay(n_panel_pieces, dim))


def adaqp_spmm_panels_workspace_bytes(n_per_tile: int, dim: int) -> int:
    out = ctypes.c_int64(0)
    _check(lib().adaqp_spmm_panels_workspace_bytes(n_per_tile, dim, ctypes.byref(out)),
           "adaqp_spmm_panels_workspace_bytes")
    return int(out.value)


def adaqp_spmm_csr_panels(panels: DevicePanels, row_begin: int, row_end: int, H: torch.Tensor, dim: int,
                          out: torch.Tensor, workspace: torch.Tensor,
                          stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr_panels(ctypes.byref(panels.c), row_begin, row_end, hp, n_cols, ldh, dim, op, ldo,
                                       _dev(workspace, torch.uint8, "workspace"), workspace.numel(),
                                       _stream(stream)), "adaqp_spmm_csr_panels")


SPMM_SEGMENTS = 8
SPMM_SEGMENTS_MOST_BYTES = 0xFFFF0000       # of H


def adaqp_plan_spmm_segments(rowptr_host: np.ndarray, row_begin: int, row_end: int, col_bounds_host: np.ndarray,
                             tile_off: np.ndarray) -> Optional[dict]:
    """Host-only.  None when the table leaves no entries, else a dict of host arrays (ptr, src, of_row) and sizes."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    bounds = np.ascontiguousarray(col_bounds_host, dtype=np.int32)
    off = np.ascontiguousarray(tile_off, dtype=np.int32)
    n_rows = max(row_end - row_begin, 0)
    if bounds.shape[0] != SPMM_TILES + 1 or off.shape != (n_rows, SPMM_TILES + 1):
        raise ValueError("col_bounds and tile_off must be adaqp_plan_spmm_tiles' outputs for this range")
    sizes = np.zeros(2, dtype=np.int64)
    args = (rowptr.ctypes.data, row_begin, row_end, bounds.ctypes.data, off.ctypes.data, sizes.ctypes.data)
    _check(lib().adaqp_plan_spmm_segments(*args, None, None, None), "adaqp_plan_spmm_segments")
    n_seg = int(sizes[0])
    if n_seg == 0:
        return None
    plan = {"n_seg": n_seg, "n_entries": int(sizes[1]), "n_rows": n_rows, "ptr": np.empty(n_seg + 1, dtype=np.int64),
            "src": np.empty(n_seg, dtype=np.int64), "of_row": np.empty((n_rows, SPMM_SEGMENTS), dtype=np.int32)}
    _check(lib().adaqp_plan_spmm_segments(*args, plan["ptr"].ctypes.data, plan["src"].ctypes.data, plan["of_row"].ctypes.data),
           "adaqp_plan_spmm_segments")
    return plan


def adaqp_spmm_segments_lines(col_bounds_host: np.ndarray) -> int:
    bounds = np.ascontiguousarray(col_bounds_host, dtype=np.int32)
    if bounds.shape[0] != SPMM_TILES + 1:
        raise ValueError("col_bounds must be an output of adaqp_plan_spmm_tiles")
    return int(lib().adaqp_spmm_segments_lines(bounds.ctypes.data))


SPMM_PIECE = np.dtype([("entry", np.int64), ("segment", np.int32), ("partial", np.int32)])


def adaqp_plan_spmm_pieces(ptr_host: np.ndarray, of_row_host: Optional[np.ndarray], dim: int, lines_per_slice: int) -> dict:
    """Host-only.  The pieces of the walk over the segments of adaqp_plan_spmm_segments (its ptr and of_row), for rows of dim columns:
    or, without of_row, over rows whose rowptr is ptr: a dict of host arrays (pieces, dest, sum_row, sum_ptr) and lines_per_slice."""
    ptr = np.ascontiguousarray(ptr_host, dtype=np.int64)
    of_row = None if of_row_host is None else np.ascontiguousarray(of_row_host, dtype=np.int32).reshape(-1, SPMM_SEGMENTS)
    sizes = np.zeros(5, dtype=np.int64)
    args = (ptr.ctypes.data, ptr.shape[0] - 1, None if of_row is None else of_row.ctypes.data,
            ptr.shape[0] - 1 if of_row is None else of_row.shape[0], dim, lines_per_slice, sizes.ctypes.data)
    _check(lib().adaqp_plan_spmm_pieces(*args, None, None, None, None), "adaqp_plan_spmm_pieces")
    plan = {"pieces": np.empty(int(sizes[0]) + 1, dtype=SPMM_PIECE), "dest": np.empty(ptr.shape[0] - 1, dtype=np.int32),
            "sum_row": np.empty(int(sizes[2]), dtype=np.int32), "sum_ptr": np.empty(int(sizes[2]) + 1, dtype=np.int32)}
    _check(lib().adaqp_plan_spmm_pieces(*args, *(plan[k].ctypes.data for k in ("pieces", "dest", "sum_row", "sum_ptr"))),
           "adaqp_plan_spmm_pieces")
    plan["lines_per_slice"], plan["waves"], plan["entries"] = lines_per_slice, int(sizes[3]), int(sizes[4])
    return plan


def adaqp_spmm_pieces_workspace_bytes(n_partials: int, dim: int) -> int:
    out = ctypes.c_int64(0)
    _check(lib().adaqp_spmm_pieces_workspace_bytes(n_partials, dim, ctypes.byref(out)), "adaqp_spmm_pieces_workspace_bytes")
    return int(out.value)


class DevicePieces:
    """Device copies of a plan of pieces over rows and the struct the C calls take.  Keeps the tensors alive."""

    def __init__(self, plan: Optional[dict], device="cuda", row_begin: int = 0):
        self.tensors = {}
        self.c = SpmmPieces() if plan is None else _device_pieces(plan, device, self.tensors, row_begin)

    def __bool__(self) -> bool:
        return self.c.n_pieces > 0


def _device_pieces(plan: dict, device, tensors: dict, row_begin: int = 0) -> SpmmPieces:
    """Uploads a plan of pieces into `tensors`, which keeps them alive, and returns the struct the C calls take."""
    for k in ("pieces", "dest", "sum_row", "sum_ptr"):
        tensors[k] = torch.from_numpy(plan[k].view(np.int32)).to(device)
    return SpmmPieces(plan["pieces"].shape[0] - 1, int(plan["sum_ptr"][-1]), plan["sum_row"].shape[0], plan["dest"].shape[0], row_begin,
                      plan["lines_per_slice"], plan["waves"], plan["entries"], 0,
                      *(tensors[k].data_ptr() for k in ("pieces", "dest", "sum_row", "sum_ptr")))


SPMM_SEGMENTS_MIN_GAIN = 2e6


def adaqp_spmm_segments_gain(rowptr_host: np.ndarray, col_host: np.ndarray, row_begin: int, row_end: int, n_cols: int, dim: int,
                             transposed: bool = False) -> float:
    """Host-only.  What segments without pieces save for these rows; the ranges of a step add up to SPMM_SEGMENTS_MIN_GAIN where they pay."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    col = np.ascontiguousarray(col_host, dtype=np.int32)
    out = ctypes.c_double(0.0)
    _check(lib().adaqp_spmm_segments_gain(rowptr.ctypes.data, col.ctypes.data, row_begin, row_end, n_cols, dim, int(transposed),
                                          ctypes.byref(out)), "adaqp_spmm_segments_gain")
    return out.value


def adaqp_spmm_pieces_rule(rowptr_host: np.ndarray, col_host: np.ndarray, row_begin: int, row_end: int, n_cols: int, dim: int,
                           transposed: bool = False, segments: bool = True):
    """Host-only.  (lines per slice of pieces over these rows, what segments save over that: the ranges of a step add up to more than 0
    where they pay).  segments=False: only the lines, of rows that list their columns in any order; the gain is -infinity."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    col = np.ascontiguousarray(col_host, dtype=np.int32)
    lines, gain = ctypes.c_int32(0), ctypes.c_double(-np.inf)
    _check(lib().adaqp_spmm_pieces_rule(rowptr.ctypes.data, col.ctypes.data, row_begin, row_end, n_cols, dim, int(transposed),
                                        ctypes.byref(lines), ctypes.byref(gain) if segments else None), "adaqp_spmm_pieces_rule")
    return lines.value, gain.value


class DeviceSegments:
    """Device copies of a segment plan, its copy of the entries and the struct the C calls take.  Keeps the tensors alive."""

    def __init__(self, plan: Optional[dict], device="cuda"):
        self.c = SpmmSegments()
        self.tensors = {}
        if plan is None:
            return
        for k in ("ptr", "src", "of_row"):
            self.tensors[k] = torch.from_numpy(plan[k]).to(device)
        self.tensors["col"] = torch.empty(plan["n_entries"], dtype=torch.int32, device=device)
        self.tensors["val"] = torch.empty(plan["n_entries"], dtype=torch.float32, device=device)
        t = self.tensors
        self.c = SpmmSegments(plan["n_seg"], plan["n_entries"], plan["n_rows"], t["ptr"].data_ptr(), t["src"].data_ptr(),
                              t["of_row"].data_ptr(), t["col"].data_ptr(), t["val"].data_ptr())
        if "pieces" in plan:
            self.c.pieces = _device_pieces(plan["pieces"], device, t)

    def __bool__(self) -> bool:
        return self.c.n_seg > 0


def adaqp_fill_spmm_segments(segments: DeviceSegments, col: torch.Tensor, val: torch.Tensor,
                             stream: Optional[torch.cuda.Stream] = None) -> None:
    _check(lib().adaqp_fill_spmm_segments(ctypes.byref(segments.c), _dev(col, torch.int32, "col"),
                                          _dev(val, torch.float32, "val"), col.numel(), _stream(stream)),
           "adaqp_fill_spmm_segments")


def adaqp_update_spmm_segments(segments: DeviceSegments, val: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    _check(lib().adaqp_update_spmm_segments(ctypes.byref(segments.c), _dev(val, torch.float32, "val"), val.numel(), _stream(stream)),
           "adaqp_update_spmm_segments")


def adaqp_spmm_segments_workspace_bytes(segments: DeviceSegments, dim: int) -> int:
    out = ctypes.c_int64(0)
    if segments.c.pieces.n_pieces > 0:
        return adaqp_spmm_pieces_workspace_bytes(segments.c.pieces.n_partials, dim)
    _check(lib().adaqp_spmm_segments_workspace_bytes(segments.c.n_seg, segments.c.n_entries, dim, ctypes.byref(out)),
           "adaqp_spmm_segments_workspace_bytes")
    return int(out.value)


def adaqp_spmm_csr_segments(segments: DeviceSegments, row_begin: int, H: torch.Tensor, dim: int, out: torch.Tensor,
                            workspace: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    """out: the whole matrix; row_begin: the first row of the range the plan was made for."""
    if row_begin < 0 or row_begin + segments.c.n_rows > out.shape[0]:
        raise ValueError("out does not have the rows of the plan from row_begin on")
    hp, n_cols, ldh = _matrix(H, "H")
    _, _, ldo = _matrix(out, "out")
    op, _, _ = _matrix(out[row_begin:], "out")
    _check(lib().adaqp_spmm_csr_segments(ctypes.byref(segments.c), hp, n_cols, ldh, dim, op, ldo,
                                         _dev(workspace, torch.uint8, "workspace"), workspace.numel(), _stream(stream)),
           "adaqp_spmm_csr_segments")


SPMM_BLOCK_ROWS = 128
SPMM_BLOCK_STEP = 32


def adaqp_plan_spmm_blocks(rowptr_host: np.ndarray, col_host: np.ndarray, row_begin: int, row_end: int, n_cols: int, dim: int,
                           min_row_len: int, tile_off: Optional[np.ndarray] = None,
                           only_if_pays_for_ld: int = 0, if_slower: bool = False, beside: bool = False) -> Optional[dict]:
    """Host-only.  None when no row of the range has min_row_len entries, else a dict of host arrays (rows, step_ptr, cols) and
    sizes.  With only_if_pays_for_ld = the pitch of H: the longest of these rows whose blocks adaqp_spmm_blocks_pay and
    (unless if_slower) adaqp_spmm_blocks_save(beside) speak for and whose table adaqp_spmm_blocks_most_steps allows, None if there are none.
    tile_off (the table of adaqp_plan_spmm_tiles for the same range) is changed in place: the rows taken are struck."""
    rowptr = np.ascontiguousarray(rowptr_host, dtype=np.int64)
    col = np.ascontiguousarray(col_host, dtype=np.int32)
    if tile_off is not None:
        if tile_off.dtype != np.int32 or not tile_off.flags.c_contiguous or \
                tile_off.shape != (max(row_end - row_begin, 0), SPMM_TILES + 1):
            raise ValueError("tile_off must be the C-contiguous int32 table of adaqp_plan_spmm_tiles for this range")
    names = ("n_rows_taken", "n_blocks", "n_pieces", "n_steps", "col_begin", "piece_width")
    degs = np.diff(rowptr[row_begin:row_end + 1]) if only_if_pays_for_ld > 0 else None
    while True:
        sizes = np.zeros(6, dtype=np.int64)
        args = (rowptr.ctypes.data, col.ctypes.data, row_begin, row_end, n_cols, dim, min_row_len, sizes.ctypes.data)
        _check(lib().adaqp_plan_spmm_blocks(*args, None, None, None, None), "adaqp_plan_spmm_blocks")
        plan = {k: int(v) for k, v in zip(names, sizes)}
        if plan["n_rows_taken"] == 0:
            return None
        if only_if_pays_for_ld <= 0:
            break
        if not lib().adaqp_spmm_blocks_pay(plan["n_rows_taken"], n_cols, only_if_pays_for_ld):
            return None
        if plan["n_steps"] <= lib().adaqp_spmm_blocks_most_steps(int(degs.sum())) and \
                (if_slower or lib().adaqp_spmm_blocks_save(int(degs[degs >= min_row_len].sum()), plan["n_steps"], dim, int(beside))):
            break
        min_row_len += min_row_len // 2 + 1                 # the longer ones fill their blocks better
    plan.update(rows=np.empty(plan["n_blocks"] * SPMM_BLOCK_ROWS, dtype=np.int32),
                step_ptr=np.empty(plan["n_blocks"] * plan["n_pieces"] + 1, dtype=np.int32),
                cols=np.empty((plan["n_steps"], SPMM_BLOCK_STEP), dtype=np.int32))
    _check(lib().adaqp_plan_spmm_blocks(*args, None if tile_off is None else tile_off.ctypes.data, plan["rows"].ctypes.data,
                                        plan["step_ptr"].ctypes.data, plan["cols"].ctypes.data), "adaqp_plan_spmm_blocks")
    return plan


def adaqp_spmm_blocks_min_row(n_cols: int) -> int:
    """Host-only.  The row length from which a row is worth a place in a block."""
    return int(lib().adaqp_spmm_blocks_min_row(n_cols))


class DeviceBlocks:
    """Device copies of a block plan, its table of coefficients and the struct the C calls take.  Keeps the tensors alive."""

    def __init__(self, plan: Optional[dict], device="cuda"):
        self.c = SpmmBlocks()
        self.tensors = {}
        if plan is None:
            return
        for k in ("rows", "step_ptr", "cols"):
            self.tensors[k] = torch.from_numpy(plan[k]).to(device)
        self.tensors["table"] = torch.empty(int(lib().adaqp_spmm_blocks_table_floats(plan["n_steps"])), dtype=torch.float32,
                                            device=device)
        t = self.tensors
        self.c = SpmmBlocks(plan["n_blocks"], plan["n_pieces"], plan["n_steps"], plan["col_begin"], plan["piece_width"],
                            t["rows"].data_ptr(), t["step_ptr"].data_ptr(), t["cols"].data_ptr(), t["table"].data_ptr())

    def __bool__(self) -> bool:
        return self.c.n_blocks > 0


def adaqp_fill_spmm_blocks(blocks: DeviceBlocks, row_begin: int, row_end: int, rowptr: torch.Tensor, col: torch.Tensor,
                           val: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    _check(lib().adaqp_fill_spmm_blocks(ctypes.byref(blocks.c), row_begin, row_end, _dev(rowptr, torch.int64, "rowptr"),
                                        _dev(col, torch.int32, "col"), _dev(val, torch.float32, "val"), col.numel(),
                                        _stream(stream)), "adaqp_fill_spmm_blocks")


def adaqp_update_spmm_blocks(blocks: DeviceBlocks, row_begin: int, row_end: int, rowptr: torch.Tensor, col: torch.Tensor,
                             val: torch.Tensor, copied: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    """copied: what val held for the entries of the rows at the time of the fill, brought up to date."""
    _check(lib().adaqp_update_spmm_blocks(ctypes.byref(blocks.c), row_begin, row_end, _dev(rowptr, torch.int64, "rowptr"),
                                          _dev(col, torch.int32, "col"), _dev(val, torch.float32, "val"), col.numel(),
                                          _dev(copied, torch.float32, "copied"), _stream(stream)), "adaqp_update_spmm_blocks")


def adaqp_spmm_blocks_workspace_bytes(blocks: DeviceBlocks, dim: int) -> int:
    out = ctypes.c_int64(0)
    _check(lib().adaqp_spmm_blocks_workspace_bytes(blocks.c.n_blocks, blocks.c.n_pieces, dim, ctypes.byref(out)),
           "adaqp_spmm_blocks_workspace_bytes")
    return int(out.value)


def adaqp_spmm_csr_blocks(blocks: DeviceBlocks, row_begin: int, row_end: int, H: torch.Tensor, dim: int, out: torch.Tensor,
                          workspace: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr_blocks(ctypes.byref(blocks.c), row_begin, row_end, hp, n_cols, ldh, dim, op, ldo,
                                       _dev(workspace, torch.uint8, "workspace"), workspace.numel(), _stream(stream)),
           "adaqp_spmm_csr_blocks")


def adaqp_spmm_csr_tiled(rowptr: torch.Tensor, col: torch.Tensor, val: torch.Tensor, row_begin: int, row_end: int,
                         H: torch.Tensor, dim: int, out: torch.Tensor, tile_off: torch.Tensor,
                         workspace: torch.Tensor, chunk_cols: int = 0,
                         stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr_tiled(_dev(rowptr, torch.int64, "rowptr"), _dev(col, torch.int32, "col"),
                                      _dev(val, torch.float32, "val"), col.numel(), row_begin, row_end,
                                      hp, n_cols, ldh, dim, op, ldo, _dev(tile_off, torch.int32, "tile_off"),
                                      chunk_cols, _dev(workspace, torch.uint8, "workspace"), workspace.numel(),
                                      _stream(stream)), "adaqp_spmm_csr_tiled")


def adaqp_assign_bits(beta_host: np.ndarray, peer_of_slot_host: np.ndarray, n_peers: int, dim: int,
                      group_size: int, lam: float, theta: np.ndarray, gamma: np.ndarray
                      ) -> Tuple[np.ndarray, np.ndarray]:
    """Host-only.  Returns (bits uint8[n], float64[3] = Eq. 9 value, variance, largest pair time)."""
    beta = np.ascontiguousarray(beta_host, dtype=np.float32)
    peer = np.ascontiguousarray(peer_of_slot_host, dtype=np.int32)
    theta = np.ascontiguousarray(theta, dtype=np.float64)
    gamma = np.ascontiguousarray(gamma, dtype=np.float64)
    if theta.shape[0] != n_peers or gamma.shape[0] != n_peers or peer.shape[0] != beta.shape[0]:
        raise ValueError("theta / gamma need n_peers entries, peer_of_slot one per beta")
    bits = np.zeros(beta.shape[0], dtype=np.uint8)
    obj = np.zeros(3, dtype=np.float64)
    _check(lib().adaqp_assign_bits(beta.shape[0], beta.ctypes.data, peer.ctypes.data, n_peers, dim, group_size,
                                   float(lam), theta.ctypes.data, gamma.ctypes.data, bits.ctypes.data,
                                   obj.ctypes.data), "adaqp_assign_bits")
    return bits, obj


def adaqp_plan_slot_of_row(n_rows: int, halo_idx_host: np.ndarray) -> np.ndarray:
    """Host-only.  Returns int32[n_rows]: the slot received into each row, -1 elsewhere."""
    halo = np.ascontiguousarray(halo_idx_host, dtype=np.int32)
    out = np.zeros(n_rows, dtype=np.int32)
    _check(lib().adaqp_plan_slot_of_row(n_rows, halo.shape[0], halo.ctypes.data, out.ctypes.data),
           "adaqp_plan_slot_of_row")
    return out


def adaqp_plan_packed_rows(n_rows: int, halo_idx_host: np.ndarray, bits_host: np.ndarray, row_offset_host: np.ndarray, dim: int,
                           packed_bytes: int) -> np.ndarray:
    """Host-only.  uint32[n_rows, 2]: place in the receive buffer and slot of each received row, 0 elsewhere."""
    halo = np.ascontiguousarray(halo_idx_host, dtype=np.int32)
    bits = np.ascontiguousarray(bits_host, dtype=np.uint8)
    offset = np.ascontiguousarray(row_offset_host, dtype=np.int64)
    if not halo.shape == bits.shape == offset.shape:
        raise ValueError("halo_idx, bits and row_offset must have one value per slot")
    out = np.zeros((n_rows, 2), dtype=np.uint32)
    _check(lib().adaqp_plan_packed_rows(n_rows, halo.shape[0], halo.ctypes.data, bits.ctypes.data, offset.ctypes.data, dim, packed_bytes,
                                        out.ctypes.data), "adaqp_plan_packed_rows")
    return out


def adaqp_spmm_csr_packed(rowptr: torch.Tensor, col: torch.Tensor, val: torch.Tensor, row_begin: int, row_end: int,
                          H: torch.Tensor, dim: int, out: torch.Tensor, slot_of_row: torch.Tensor,
                          packed: torch.Tensor, params: torch.Tensor, bits: torch.Tensor, row_offset: torch.Tensor,
                          workspace: torch.Tensor, nnz_range: int = -1,
                          stream: Optional[torch.cuda.Stream] = None) -> None:
    hp, n_cols, ldh = _matrix(H, "H")
    op, _, ldo = _matrix(out, "out")
    _check(lib().adaqp_spmm_csr_packed(_dev(rowptr, torch.int64, "rowptr"), _dev(col, torch.int32, "col"),
                                       _dev(val, torch.float32, "val"), col.numel(), row_begin, row_end, nnz_range,
                                       hp, n_cols, ldh, dim, op, ldo,
                                       _dev(slot_of_row, torch.int32, "slot_of_row"),
                                       _dev(packed, torch.uint8, "packed"), packed.numel(),
                                       _dev(params, torch.float32, "params"), _dev(bits, torch.uint8, "bits"),
                                       _dev(row_offset, torch.int64, "row_offset"), bits.shape[0],
                                       _dev(workspace, torch.uint8, "workspace"), workspace.numel(),
                                       _stream(stream)),
           "adaqp_spmm_csr_packed")


def adaqp_layer_step(desc: LayerDesc) -> None:
    _check(lib().adaqp_layer_step(ctypes.byref(desc)), "adaqp_layer_step")


def adaqp_probe_quantize_pack(feat: torch.Tensor, dim: int, send_idx: torch.Tensor, bits: torch.Tensor,
                              row_offset: torch.Tensor, packed: torch.Tensor, params: torch.Tensor,
                              stream: Optional[torch.cuda.Stream] = None) -> None:
    """Measurement aid (include/adaqp_probe.h): the no-compute twin of adaqp_quantize_pack."""
    fp, n_rows, ld = _matrix(feat, "feat")
    _check(lib().adaqp_probe_quantize_pack(fp, n_rows, ld, dim, _dev(send_idx, torch.int32, "send_idx"),
                                           _dev(bits, torch.uint8, "bits"),
                                           _dev(row_offset, torch.int64, "row_offset"), send_idx.shape[0],
                                           _dev(packed, torch.uint8, "packed"), packed.numel(),
                                           _dev(params, torch.float32, "params"), _stream(stream)),
           "adaqp_probe_quantize_pack")


def adaqp_probe_unpack_dequant_add(packed: torch.Tensor, params: torch.Tensor, bits: torch.Tensor,
                                   row_offset: torch.Tensor, dst_idx: torch.Tensor, seg_order: torch.Tensor,
                                   seg_ptr: torch.Tensor, dim: int, grad: torch.Tensor,
                                   stream: Optional[torch.cuda.Stream] = None) -> None:
    """Measurement aid (include/adaqp_probe.h): the no-compute twin of adaqp_unpack_dequant_add."""
    gp, n_rows, ld = _matrix(grad, "grad")
    _check(lib().adaqp_probe_unpack_dequant_add(_dev(packed, torch.uint8, "packed"), packed.numel(),
                                                _dev(params, torch.float32, "params"),
                                                _dev(bits, torch.uint8, "bits"),
                                                _dev(row_offset, torch.int64, "row_offset"),
                                                _dev(dst_idx, torch.int32, "dst_idx"), dst_idx.shape[0],
                                                _dev(seg_order, torch.int32, "seg_order"),
                                                _dev(seg_ptr, torch.int64, "seg_ptr"), seg_ptr.shape[0] - 1,
                                                dim, gp, n_rows, ld, _stream(stream)),
           "adaqp_probe_unpack_dequant_add")


def adaqp_probe_stream(src: torch.Tensor, dst: torch.Tensor, nbytes: int, write_side: int,
                       stream: Optional[torch.cuda.Stream] = None) -> None:
    """Measurement aid (include/adaqp_probe.h): a plain stream over nbytes bytes of src (write_side 0), of dst
    (1), or of dst read and written back in place (2)."""
    write_side = int(write_side)
    big, small = (dst, src) if write_side else (src, dst)
    if big.numel() * big.element_size() < nbytes or small.numel() * small.element_size() < nbytes // 8 + 4096:
        raise ValueError("adaqp_probe_stream: a buffer is smaller than the stream")
    if not (src.is_cuda and dst.is_cuda and src.is_contiguous() and dst.is_contiguous()):
        raise TypeError("adaqp_probe_stream needs contiguous device tensors")
    _check(lib().adaqp_probe_stream(src.data_ptr(), dst.data_ptr(), nbytes, write_side, _stream(stream)),
           "adaqp_probe_stream")


def adaqp_probe_xcd_of_workgroup(n_workgroups: int, device="cuda:0",
                                 stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """Measurement aid (include/adaqp_probe.h): the XCD each workgroup of a 1-D grid runs on (int32 device tensor)."""
    out = torch.full((max(n_workgroups, 1),), -1, dtype=torch.int32, device=device)
    _check(lib().adaqp_probe_xcd_of_workgroup(out.data_ptr(), n_workgroups, _stream(stream)),
           "adaqp_probe_xcd_of_workgroup")
    return out[:n_workgroups]
