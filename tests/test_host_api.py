"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, and its host logic
(layout planning, argument validation that happens before any launch) behaves as the header says."""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_2306_01381_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    names = set()
    inc = os.path.join(ROOT, "include")
    for header in sorted(os.listdir(inc)):
        if header.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, header)).read(), flags=re.S)
            names |= set(re.findall(r"\b(adaqp_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = _declared_symbols()
    assert len(names) >= 10
    for n in names:
        assert hasattr(L, n), n
    assert set(names) == set(B.EXPORTS)
    assert B.adaqp_version() >= 100
    assert L.adaqp_strerror(B.ESIZE).decode().startswith("buffer")


def test_row_stride():
    assert B.adaqp_row_stride(602, 2) == 152 and B.adaqp_row_stride(602, 4) == 304
    assert B.adaqp_row_stride(602, 8) == 604 and B.adaqp_row_stride(1, 2) == 4
    assert B.adaqp_row_stride(256, 2) == 64
    assert B.adaqp_row_stride(0, 2) == -1 and B.adaqp_row_stride(8, 3) == -1


def test_plan_layout_matches_oracle(oracle):
    rng = np.random.default_rng(4)
    for dim in (1, 5, 128, 300, 602, 4100):
        for n, n_peers in ((0, 2), (1, 1), (37, 3), (500, 7)):
            peer = np.sort(rng.integers(0, n_peers, size=n)).astype(np.int32)
            bits = rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=n)
            got = B.adaqp_plan_layout(dim, bits, peer, n_peers)
            want = oracle.plan_layout(dim, bits, peer, n_peers)
            for g, w in zip(got, want):
                assert np.array_equal(g, w)


def test_plan_layout_errors():
    with pytest.raises(B.AdaqpError) as e:
        B.adaqp_plan_layout(8, np.array([2, 5], np.uint8), np.array([0, 0], np.int32), 1)
    assert e.value.status == B.EBITS
    with pytest.raises(B.AdaqpError) as e:
        B.adaqp_plan_layout(8, np.array([2, 2], np.uint8), np.array([1, 0], np.int32), 2)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_layout(0, np.array([2], np.uint8), np.array([0], np.int32), 1)
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_layout(8, np.array([2], np.uint8), np.array([3], np.int32), 3)


def test_argument_errors_are_caught_before_any_launch():
    L = B.lib()
    one = ctypes.c_void_p(256)          # a non-NULL, aligned dummy; never dereferenced on these paths
    # zero counts are successful no-ops
    assert L.adaqp_quantize_pack(None, 0, 8, 8, None, None, None, 0, 0, None, 0, None, None) == B.OK
    assert L.adaqp_unpack_dequant(None, 0, None, None, None, None, None, 0, 8, None, 0, 8, None) == B.OK
    assert L.adaqp_spmm_csr(None, None, None, 0, 3, 3, -1, None, 0, 8, 8, None, 8, None, 0, None) == B.OK
    # bad shapes
    assert L.adaqp_quantize_pack(one, 4, 7, 8, one, one, one, 1, 0, one, 64, one, None) == B.EINVAL   # ld < dim
    assert L.adaqp_quantize_pack(one, 4, 8, 0, one, one, one, 1, 0, one, 64, one, None) == B.EINVAL   # dim 0
    assert L.adaqp_quantize_pack(one, 4, 8, 8, one, one, one, -1, 0, one, 64, one, None) == B.EINVAL  # n < 0
    assert L.adaqp_quantize_pack(None, 4, 8, 8, one, one, one, 1, 0, one, 64, one, None) == B.EINVAL  # NULL
    assert L.adaqp_unpack_dequant(one, 64, one, one, one, one, None, 1, 8, None, 4, 8, None) == B.EINVAL
    assert L.adaqp_unpack_dequant(one, 64, one, one, one, one, None, 1, 8, one, 4, 4, None) == B.EINVAL  # ld < dim
    assert L.adaqp_spmm_csr(one, one, one, 5, 2, 1, -1, one, 4, 8, 8, one, 8, one, 1 << 20, None) == B.EINVAL
    assert L.adaqp_spmm_csr(one, one, one, 5, 0, 2, -1, one, 4, 4, 8, one, 8, one, 1 << 20, None) == B.EINVAL
    # workspace too small
    assert L.adaqp_spmm_csr(one, one, one, 5, 0, 2, -1, one, 4, 8, 8, one, 8, one, 16, None) == B.ESIZE
    assert L.adaqp_layer_step(None) == B.EINVAL
    d = B.LayerDesc()
    d.direction = 7
    assert L.adaqp_layer_step(ctypes.byref(d)) == B.EINVAL
    # panels: nothing to do is fine, anything inconsistent is refused on the host
    assert L.adaqp_spmm_csr_panels(None, 0, 4, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.EINVAL
    none = B.SpmmPanels()
    assert L.adaqp_spmm_csr_panels(ctypes.byref(none), 0, 4, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.OK
    some = B.SpmmPanels(1, 1, 1, 1, 256, 256, 256, 256, 256, 256)
    assert L.adaqp_spmm_csr_panels(ctypes.byref(some), 0, 4, one, 8, 32, 8, one, 32, one, 16, None) == B.ESIZE
    assert L.adaqp_spmm_csr_panels(ctypes.byref(some), 0, 4, one, 8, 24, 8, one, 32, one, 1 << 20, None) == B.EINVAL  # pitch
    assert L.adaqp_spmm_csr_panels(ctypes.byref(some), 0, 4, one, 8, 32, 8, one, 32, None, 1 << 20, None) == B.EINVAL
    assert L.adaqp_spmm_csr_panels(ctypes.byref(some), 4, 0, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.EINVAL
    holes = B.SpmmPanels(1, 1, 1, 1, 256, 0, 256, 256, 256, 256)                    # an array missing
    assert L.adaqp_spmm_csr_panels(ctypes.byref(holes), 0, 4, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.EINVAL
    many = B.SpmmPanels(1, 1, 1, 9, 256, 256, 256, 256, 256, 256)                   # more pieces than piece slots
    assert L.adaqp_spmm_csr_panels(ctypes.byref(many), 0, 4, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.EINVAL
    bad = B.SpmmPanels(-1, 0, 0, 0, 0, 0, 0, 0, 0, 0)
    assert L.adaqp_spmm_csr_panels(ctypes.byref(bad), 0, 4, one, 8, 32, 8, one, 32, one, 1 << 20, None) == B.EINVAL


def test_layer_step_refuses_plans_before_it_queues_anything():
    """Segments or blocks that the aggregation would refuse: the codes of its checks, where a step that has begun could only fail to
    launch (no GPU here) or leave its messages queued."""
    L = B.lib()

    def desc(**kw):
        d = B.LayerDesc(direction=B.FORWARD, schedule=B.SERIAL, rowptr_dev=256, col_dev=256, val_dev=256, nnz=100, overlap_begin=0,
                        overlap_end=4, dependent_begin=4, dependent_end=4, overlap_nnz=100, feat_dev=256, n_feat_rows=8, ld=32, dim=32,
                        out_dev=256, ldo=32, tile_off_overlap_dev=256, workspace_overlap_dev=256, workspace_overlap_bytes=1 << 30)
        for k, v in kw.items():
            setattr(d, k, v)
        return L.adaqp_layer_step(ctypes.byref(d))

    def segments(n_rows=4, ptr=256):
        return B.SpmmSegments(3, 100, n_rows, ptr, 256, 256, 256, 256)

    def blocks(n_blocks=1, cols=256):
        return B.SpmmBlocks(n_blocks, 8, 8, 0, 1, 256, 256, cols, 256)

    assert desc(segments_overlap=segments(n_rows=5)) == B.EINVAL         # of another range
    assert desc(segments_overlap=segments(), segments_dependent=segments()) == B.EINVAL
    for plan in ({"segments_overlap": segments()}, {"blocks_overlap": blocks()}):
        assert desc(**plan, ld=40) == B.EINVAL                          # rows that do not start on lines
        assert desc(**plan, ldo=40) == B.EINVAL
        assert desc(**plan, feat_dev=64) == B.EINVAL
        assert desc(**plan, out_dev=64) == B.EINVAL
        assert desc(**plan, workspace_overlap_dev=128) == B.EINVAL
        assert desc(**plan, n_feat_rows=1 << 26) == B.ESIZE             # H of 2^33 bytes
    assert desc(segments_overlap=segments(ptr=260)) == B.EINVAL
    # a range without rows reads no workspace
    assert desc(overlap_end=0, dependent_begin=0, dependent_end=0, blocks_overlap=blocks(), workspace_overlap_dev=128) == B.OK
    assert desc(blocks_overlap=blocks(cols=264)) == B.EINVAL
    assert desc(blocks_overlap=blocks(n_blocks=1 << 17)) == B.ESIZE     # more workgroups than a launch has
    assert not L.adaqp_spmm_blocks_pay(1 << 24, 1000, 32) and L.adaqp_spmm_blocks_pay(1 << 22, 1000, 32)


def test_segments_of_rows_that_the_output_does_not_have():
    """A first row from which the plan's rows do not fit the matrix is refused before anything is launched."""
    import torch
    from types import SimpleNamespace
    plan = SimpleNamespace(c=B.SpmmSegments(3, 100, 6, 256, 256, 256, 256, 256))
    out, ws = torch.zeros(8, 32), torch.zeros(256, dtype=torch.uint8)
    for row_begin in (-1, 3, 8, 9):
        with pytest.raises(ValueError):
            B.adaqp_spmm_csr_segments(plan, row_begin, torch.zeros(8, 32), 32, out, ws)
    with pytest.raises(TypeError):                                     # the rows fit: a host matrix is refused next
        B.adaqp_spmm_csr_segments(plan, 2, torch.zeros(8, 32), 32, out, ws)


def test_workspace_query():
    assert B.adaqp_spmm_workspace_bytes(0, 0, 8) == 0
    small = B.adaqp_spmm_workspace_bytes(2000, 20000, 128)
    big = B.adaqp_spmm_workspace_bytes(58000, 28_000_000, 602)
    assert small % 256 == 0 and big % 256 == 0 and 0 < small < big < (1 << 30)
    with pytest.raises(B.AdaqpError):
        B.adaqp_spmm_workspace_bytes(-1, 0, 8)


def test_plan_recv_order():
    rng = np.random.default_rng(3)
    halo = rng.permutation(5000)[:700].astype(np.int32) + 100
    order = B.adaqp_plan_recv_order(halo)
    assert order.dtype == np.int32 and sorted(order.tolist()) == list(range(700))
    assert np.all(np.diff(halo[order]) > 0)
    assert np.array_equal(order, np.argsort(halo, kind="stable"))
    assert B.adaqp_plan_recv_order(np.zeros(0, np.int32)).size == 0
    # ties keep slot order
    assert B.adaqp_plan_recv_order(np.array([5, 1, 5, 1], np.int32)).tolist() == [1, 3, 0, 2]


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 5000])
@pytest.mark.parametrize("span", [1, 5, 2_000, 3_000_000, 2**32])
def test_plan_recv_order_ranges(n, span):
    """Few values, a partition's rows, values all over the range of the type, negative ones among them; every way the
    planner sorts them against a stable comparison sort."""
    rng = np.random.default_rng(n + span)
    dst = (rng.integers(0, span, size=n) - span // 2).astype(np.int32)
    want = np.argsort(dst, kind="stable")
    assert np.array_equal(B.adaqp_plan_recv_order(dst), want)
    assert np.array_equal(B.adaqp_plan_recv_order(dst[want]), np.arange(n))
    order, seg_ptr = B.adaqp_plan_recv_segments(dst)
    assert np.array_equal(order, want)
    assert np.array_equal(seg_ptr, np.append(np.flatnonzero(np.diff(dst[want], prepend=dst[want[0]].astype(np.int64) - 1)), n))


@pytest.mark.parametrize("span", [12_000_000, 2**31])
def test_plan_recv_order_without_room(span):
    """Scratch that cannot be had is no error, and no exception leaves the library."""
    code = f"""
import resource, numpy as np
from paper_2306_01381_amd import binding as B
dst = np.random.default_rng(1).integers(0, {span}, size=4_000_000).astype(np.int32)
want = np.argsort(dst, kind="stable")
B.adaqp_plan_recv_order(dst[:1000])
pages = int(open("/proc/self/statm").read().split()[0])
limit = pages * resource.getpagesize() + (28 << 20)     # the result fits, counters or keys do not
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
assert np.array_equal(B.adaqp_plan_recv_order(dst), want)
print("same order")
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert done.returncode == 0 and "same order" in done.stdout, done.stderr[-2000:]


def test_spmm_workspace_of_few_rows():
    """One carry slot per 32 path steps and no more: the widest rows that fit the built-in scratch of the call without a
    workspace."""
    for n_rows, nnz, items in ((1, 5, 1), (1, 31, 1), (2, 31, 2), (40, 60, 4), (40, 100, 5)):
        for dim in (1, 33, 4096):
            ld = (dim + 31) // 32 * 32
            assert B.adaqp_spmm_workspace_bytes(n_rows, nnz, dim) == \
                (items * 4 + 255) // 256 * 256 + (items * ld * 4 + 255) // 256 * 256
    assert B.adaqp_spmm_workspace_bytes(1, 5, 16_000_000) <= B.SPMM_NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("n,peers,halo", [(0, 3, "rising"), (1, 1, "none"), (257, 1, "rising"), (1000, 7, "rising"), (1000, 7, "equal"), (1000, 4, "any"),
                                          (3000, 300, "any"), (999, 5, "none")])
def test_plan_send(n, peers, halo):
    """The layout, the caller's arrays in its order, and the visiting order of the received rows: those of the single calls."""
    rng = np.random.default_rng(n + peers)
    bits = rng.choice(np.array([2, 4, 8], np.uint8), n)
    peer = np.sort(rng.integers(0, peers, n)).astype(np.int32)
    send = rng.integers(-5, 1 << 20, n + 3)
    rows = {"rising": np.cumsum(rng.integers(1, 4, n)), "equal": np.cumsum(rng.integers(0, 2, n)), "any": rng.integers(0, 1 << 30, n), "none": None}[halo]
    plan = B.adaqp_plan_send(37, bits, peer, peers, send, rows)
    perm, off, ptr = B.adaqp_plan_layout(37, bits, peer, peers)
    want = {"perm": perm, "row_offset": off, "peer_byte_ptr": ptr, "send_idx": send[perm].astype(np.int32), "bits": bits[perm]}
    if rows is not None:
        want["halo_idx"] = rows[perm].astype(np.int32)
        want["recv_order"] = B.adaqp_plan_recv_order(want["halo_idx"])
        assert np.array_equal(want["recv_order"], np.argsort(want["halo_idx"], kind="stable"))
    for name, values in want.items():
        assert plan[name].dtype == values.dtype and np.array_equal(plan[name], values), name
    for name, (begin, size, dtype) in plan["at"].items():               # what is uploaded
        assert begin % 256 == 0 and np.array_equal(plan["blob"][begin:begin + size].view(dtype), want[name]), name
    assert ("halo_idx" in plan) == (rows is not None)
    if n:
        for wrong in (dict(bits=np.full(n, 3, np.uint8)), dict(peer=peer[::-1] - 1), dict(peer=peer + peers)):
            with pytest.raises(B.AdaqpError):
                B.adaqp_plan_send(37, wrong.get("bits", bits), wrong.get("peer", peer), peers, send, rows)


@pytest.mark.parametrize("sizes", [[63, 64, 65, 0, 66, 67, 1, 0, 0, 255, 256, 257], [0, 0, 64], [1] * 300, [128, 0]])
def test_plan_layout_of_small_and_large_peers(sizes):
    """Peers whose slots are placed in one part and in four, peers without any, and ends that are looked for near the beginning."""
    n_peers = len(sizes)
    peer = np.repeat(np.arange(n_peers, dtype=np.int32), sizes)
    rng = np.random.default_rng(peer.size)
    bits = rng.choice(np.array([2, 4, 8], np.uint8), peer.size)
    perm, off, ptr = B.adaqp_plan_layout(19, bits, peer, n_peers)
    want = np.lexsort((np.arange(peer.size), bits, peer))
    stride = np.array([B.lib().adaqp_row_stride(19, int(b)) for b in bits[want]], dtype=np.int64)
    assert np.array_equal(perm, want) and np.array_equal(off, np.cumsum(stride) - stride)
    ends = np.concatenate([[0], np.cumsum(stride)])
    assert np.array_equal(ptr, ends[np.concatenate([[0], np.cumsum(sizes)])])


def test_plan_recv_segments():
    dst = np.array([7, 3, 7, 9, 3, 3], dtype=np.int32)
    order, seg_ptr = B.adaqp_plan_recv_segments(dst)
    assert order.tolist() == [1, 4, 5, 0, 2, 3]              # by destination, slot order inside
    assert seg_ptr.tolist() == [0, 3, 5, 6]
    order, seg_ptr = B.adaqp_plan_recv_segments(np.zeros(0, np.int32))
    assert order.size == 0 and seg_ptr.tolist() == [0]
    rng = np.random.default_rng(8)
    dst = rng.integers(0, 300, size=2000).astype(np.int32)
    order, seg_ptr = B.adaqp_plan_recv_segments(dst)
    assert sorted(order.tolist()) == list(range(2000))
    assert np.all(np.diff(dst[order]) >= 0)
    assert len(seg_ptr) - 1 == len(np.unique(dst))
    for g in range(len(seg_ptr) - 1):
        seg = order[seg_ptr[g]: seg_ptr[g + 1]]
        assert len(set(dst[seg].tolist())) == 1 and np.all(np.diff(seg) > 0)


def test_plan_slot_of_row():
    halo = np.array([7, 3, 9, 4], dtype=np.int32)
    m = B.adaqp_plan_slot_of_row(10, halo)
    assert m.dtype == np.int32 and m.tolist() == [-1, -1, -1, 1, 3, -1, -1, 0, -1, 2]
    assert B.adaqp_plan_slot_of_row(3, np.zeros(0, np.int32)).tolist() == [-1, -1, -1]
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_slot_of_row(10, np.array([1, 1], dtype=np.int32))       # a row listed twice
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_slot_of_row(10, np.array([10], dtype=np.int32))         # out of range


def test_plan_spmm_tiles():
    rng = np.random.default_rng(3)
    n_rows, n_cols = 40, 100
    rowptr = np.zeros(n_rows + 1, dtype=np.int64)
    cols = []
    for r in range(n_rows):
        d = int(rng.integers(0, 30)) if r % 3 else int(rng.integers(64, 100))      # short and long rows
        cols.append(np.sort(rng.choice(n_cols, size=d, replace=False)))
        rowptr[r + 1] = rowptr[r] + d
    col = np.concatenate(cols).astype(np.int32)
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
    assert bounds.shape == (B.SPMM_TILES + 1,) and off.shape == (n_rows, B.SPMM_TILES + 1)
    assert bounds[0] == 0 and bounds[-1] == col.max() + 1 and np.all(np.diff(bounds) >= 0)
    def want_row(r, first_row, c, bnd):
        if len(c) >= B.SPMM_TILED_SHORT_ROW:
            return [int(np.count_nonzero(c < b)) for b in bnd]
        home = (r - first_row) % B.SPMM_TILES                      # a short row stays whole, in one tile
        return [0 if t <= home else len(c) for t in range(B.SPMM_TILES + 1)]

    for r in range(n_rows):
        assert off[r].tolist() == want_row(r, 0, col[rowptr[r]: rowptr[r + 1]], bounds)
    per_tile = np.array([np.count_nonzero((col >= bounds[t]) & (col < bounds[t + 1])) for t in range(B.SPMM_TILES)])
    uses = np.bincount(col, minlength=n_cols)
    assert per_tile.sum() == len(col)
    assert np.all(np.abs(per_tile - len(col) / B.SPMM_TILES) <= uses.max() + 1)      # equal up to one column's uses
    # a sub-range is planned from its own entries and indexed from its first row
    b2, off2 = B.adaqp_plan_spmm_tiles(rowptr, col, 10, 25, n_cols)
    assert off2.shape == (15, B.SPMM_TILES + 1)
    for r in (12, 13, 14, 15):
        assert off2[r - 10].tolist() == want_row(r, 10, col[rowptr[r]: rowptr[r + 1]], b2)
    # empty range, empty graph
    b3, off3 = B.adaqp_plan_spmm_tiles(rowptr, col, 5, 5, n_cols)
    assert off3.shape == (0, B.SPMM_TILES + 1) and b3[-1] == 0
    assert B.adaqp_spmm_tiled_workspace_bytes(10, 602) == 8 * 10 * 608 * 4
    assert B.adaqp_spmm_tiled_pays(28000, 12_763_658) and B.adaqp_spmm_tiled_pays(30000, 15_478_947)   # c1
    assert not B.adaqp_spmm_tiled_pays(306000, 7_680_000) and not B.adaqp_spmm_tiled_pays(0, 0)          # c2, empty
    # chunk width: 128 columns while the widest column range x 512 B stays within about 5 MB
    even = np.arange(9, dtype=np.int32)
    assert B.adaqp_spmm_tiled_chunk_cols(even * 7000, 602) == 128
    assert B.adaqp_spmm_tiled_chunk_cols(even * 13000, 602) == 64
    assert B.adaqp_spmm_tiled_chunk_cols(even * 7000, 64) == 64
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_tiles(np.array([0, 2], np.int64), np.array([5, 5], np.int32), 0, 1, 8)   # repeated column


def _panel_csr(seed, n_rows=90, n_cols=300):
    rng = np.random.default_rng(seed)
    rowptr = np.zeros(n_rows + 1, dtype=np.int64)
    cols = []
    for r in range(n_rows):
        d = int(rng.integers(0, 20)) if r % 2 else int(rng.integers(40, 200))           # short and long rows
        cols.append(np.sort(rng.choice(n_cols, size=d, replace=False)))
        rowptr[r + 1] = rowptr[r] + d
    col = np.concatenate(cols).astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    val[val == 0] = 1.0
    return rowptr, col, val


def _decode_panels(plan, n_cols):
    """Dense [n_panels * 32, n_cols] matrix a panel plan stands for, every piece visited once through the
    per-panel piece lists; also the tile of every piece."""
    dense = np.zeros((plan["n_panels"] * B.SPMM_PANEL_ROWS, n_cols), dtype=np.float64)
    npt = plan["n_per_tile"]
    seen = set()
    for p in range(plan["n_panels"]):
        ids = plan["panel_piece"][plan["panel_piece_ptr"][p]: plan["panel_piece_ptr"][p + 1]]
        assert np.all(np.diff(ids) > 0)                                 # ascending: the summation order
        for pid in ids:
            assert pid not in seen
            seen.add(int(pid))
            g0, g1 = plan["piece"][pid // npt, pid % npt]
            assert 0 <= g0 < g1 <= plan["n_groups"]
            for g in range(g0, g1):
                for u in range(4):
                    for h in range(2):
                        c = plan["pcol"][g, h, u]
                        dense[p * 32: p * 32 + 32, c] += plan["palpha"][g, 32 * h: 32 * h + 32, u]
    return dense, seen


def test_plan_spmm_panels():
    n_cols = 300
    rowptr, col, val = _panel_csr(11, n_cols=n_cols)
    n_rows = len(rowptr) - 1
    for (rb, re, min_len, piece_cols) in ((0, n_rows, 40, 16), (7, 61, 100, 8), (0, n_rows, 150, 1024)):
        bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        off0 = off.copy()
        plan = B.adaqp_plan_spmm_panels(rowptr, col, val, rb, re, n_cols, bounds, off, min_len, piece_cols)
        deg = np.diff(rowptr)
        want_rows = [r for r in range(rb, re) if deg[r] >= min_len]
        want_rows.sort(key=lambda r: (-deg[r], r))
        assert plan["n_rows_taken"] == len(want_rows) and plan["n_panels"] == (len(want_rows) + 31) // 32
        rows = plan["panel_rows"]
        assert rows[: len(want_rows)].tolist() == want_rows and np.all(rows[len(want_rows):] == -1)
        dense, seen = _decode_panels(plan, n_cols)
        assert len(seen) == plan["n_panel_pieces"]
        for k, r in enumerate(rows):
            want = np.zeros(n_cols)
            if r >= 0:
                want[col[rowptr[r]: rowptr[r + 1]]] = val[rowptr[r]: rowptr[r + 1]]
            assert np.array_equal(dense[k], want), (k, r)
        # pieces of tile t stay inside the tile's column range (the last tile takes the rest), within piece_cols
        npt = plan["n_per_tile"]
        used = 0
        for t in range(B.SPMM_TILES):
            for i in range(npt):
                g0, g1 = plan["piece"][t, i]
                if g0 == g1:
                    continue
                used += 1
                assert (g1 - g0) * 8 <= piece_cols
                c = plan["pcol"][g0:g1].reshape(-1)
                assert c.min() >= bounds[t] and (t == B.SPMM_TILES - 1 or c.max() < bounds[t + 1])
        assert used == plan["n_panel_pieces"]
        # the pieces of one (panel, tile): as few as piece_cols allows, equal in size to within one group
        sizes = {}
        for p_ in range(plan["n_panels"]):
            for pid in plan["panel_piece"][plan["panel_piece_ptr"][p_]: plan["panel_piece_ptr"][p_ + 1]]:
                g0, g1 = plan["piece"][pid // npt, pid % npt]
                sizes.setdefault((p_, int(pid) // npt), []).append(int(g1 - g0))
        for key, sz in sizes.items():
            assert max(sz) - min(sz) <= 1, (key, sz)
            assert len(sz) == -(-sum(sz) // (piece_cols // 8)), (key, sz)
        # the rows taken are struck from the tile table, the others are untouched
        taken = np.zeros(re - rb, dtype=bool)
        taken[np.array(want_rows, dtype=np.int64) - rb] = True
        assert np.all(off[taken] == -1) and np.array_equal(off[~taken], off0[~taken])
    # nothing long enough: no plan, table untouched
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
    off0 = off.copy()
    assert B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, off, 1000) is None
    assert np.array_equal(off, off0)
    assert B.adaqp_spmm_panels_workspace_bytes(218, 602) == 8 * 218 * 32 * 608 * 4
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, None, 40, 12)     # piece_cols % 8
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, None, 0, 16)      # min_row_len < 1
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_panels(np.array([0, 2], np.int64), np.array([5, 5], np.int32), np.ones(2, np.float32),
                                 0, 1, 8, np.zeros(9, np.int32), None, 1, 8)                    # repeated column


def test_plan_spmm_panels_random_graphs():
    """Seeded sweep: whatever the shape, the plan decodes back to exactly the rows it took."""
    rng = np.random.default_rng(2024)
    for case in range(12):
        n_rows = int(rng.choice([1, 5, 33, 64, 130]))
        n_cols = int(rng.choice([1, 7, 8, 9, 40, 257]))
        degs = rng.integers(0, n_cols + 1, size=n_rows)
        if case % 3 == 0:
            degs[:] = n_cols                                            # dense
        rowptr = np.zeros(n_rows + 1, dtype=np.int64)
        cols = []
        for r in range(n_rows):
            cols.append(np.sort(rng.choice(n_cols, size=int(degs[r]), replace=False)))
            rowptr[r + 1] = rowptr[r] + degs[r]
        col = np.concatenate(cols).astype(np.int32)
        val = (rng.standard_normal(len(col)) + 3.0).astype(np.float32)  # never zero
        rb = int(rng.integers(0, n_rows))
        re = int(rng.integers(rb, n_rows + 1))
        min_len = int(rng.choice([1, 2, 5, 30]))
        piece_cols = int(rng.choice([8, 16, 64]))
        bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        plan = B.adaqp_plan_spmm_panels(rowptr, col, val, rb, re, n_cols, bounds, off, min_len, piece_cols)
        want_rows = [r for r in range(rb, re) if degs[r] >= min_len]
        if not want_rows:
            assert plan is None, case
            continue
        assert sorted(plan["panel_rows"][plan["panel_rows"] >= 0].tolist()) == want_rows, case
        dense, seen = _decode_panels(plan, n_cols)
        assert len(seen) == plan["n_panel_pieces"], case
        for k, r in enumerate(plan["panel_rows"]):
            want = np.zeros(n_cols)
            if r >= 0:
                want[col[rowptr[r]: rowptr[r + 1]]] = val[rowptr[r]: rowptr[r + 1]]
            assert np.array_equal(dense[k], want), (case, k, r)


@pytest.mark.parametrize("n_rows,n_cols", [(1, 1), (60, 500), (90, 90_000)])
def test_plan_spmm_segments(n_rows, n_cols):
    """The segments of a row, in group order, are its entries in order; nothing of rows struck from the table."""
    rng = np.random.default_rng(n_cols)
    degs = np.minimum(rng.integers(0, 400, size=n_rows), n_cols)
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n_cols, size=d, replace=False)) for d in degs] or [[]]).astype(np.int32)
    for rb, re in ((0, n_rows), (n_rows // 2, n_rows)):
        bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        struck = np.arange(re - rb) % 5 == 2
        off[struck] = -1
        plan = B.adaqp_plan_spmm_segments(rowptr, rb, re, bounds, off)
        if plan is None:
            assert degs[rb:re][~struck].sum() == 0
            continue
        assert plan["ptr"][0] == 0 and plan["ptr"][-1] == plan["n_entries"] == degs[rb:re][~struck].sum()
        lengths = np.diff(plan["ptr"])
        assert np.all(lengths > 0) and plan["n_seg"] == (plan["of_row"] >= 0).sum()
        assert np.array_equal(np.sort(plan["of_row"][plan["of_row"] >= 0]), np.arange(plan["n_seg"]))
        for r in range(re - rb):
            mine = plan["of_row"][r][plan["of_row"][r] >= 0]
            if struck[r]:
                assert plan["of_row"][r][0] == -2 and mine.size == 0
                continue
            at = np.concatenate([np.arange(plan["src"][s], plan["src"][s] + lengths[s]) for s in mine] or [[]])
            assert np.array_equal(at, np.arange(rowptr[rb + r], rowptr[rb + r + 1])) and np.all(np.diff(mine) > 0)
        # a group's columns: what tiles that can be joined span
        if n_cols > 50_000:
            assert np.unique(np.nonzero(plan["of_row"] >= 0)[1]).size > 1
    with pytest.raises(B.AdaqpError):
        bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
        off[0, -1] += 1                                                # a table that disagrees with rowptr
        B.adaqp_plan_spmm_segments(rowptr, 0, n_rows, bounds, off)


def test_plan_packed_rows():
    """Place and slot of each received row; nothing where the width or the place is not one."""
    halo, bits = np.array([9, 2, 5, 7, 3], np.int32), np.array([8, 2, 4, 5, 8], np.uint8)
    offset = np.array([0, 100, 104, 200, 998], np.int64)                # dim 100: 100, 28 and 52 bytes; the last does not fit
    got = B.adaqp_plan_packed_rows(12, halo, bits, offset, 100, 1_000)
    want = np.zeros((12, 2), np.uint32)
    want[9], want[2], want[5] = (0 | 3, 0), (100 | 1, 1), (104 | 2, 2)
    assert np.array_equal(got, want)
    for rows, idx in ((4, halo), (12, np.array([9, 2, 5, 9, 3], np.int32)), (12, np.array([9, 2, 5, -1, 3], np.int32))):
        with pytest.raises(B.AdaqpError):                              # rows that there are not, one received twice
            B.adaqp_plan_packed_rows(rows, idx, bits, offset, 100, 1_000)
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_packed_rows(12, halo, bits, offset, 100, 0xFFFF0000)


@pytest.mark.parametrize("n_rows,n_cols,mean,transposed", [(300, 50, 30, False), (3_000, 9_000, 90, True), (4_000, 90_000, 200, False),
                                                           (30_000, 20, 12, False)])
def test_spmm_pieces_rule(n_rows, n_cols, mean, transposed):
    """The stated weights: lines that cost least, and what segments save over them."""
    rng = np.random.default_rng(mean)
    degs = np.minimum((rng.pareto(1.2, size=n_rows) * mean / 3).astype(np.int64), n_cols)
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n_cols, size=d, replace=False)) for d in degs]).astype(np.int32)
    for rb, re in ((0, n_rows), (n_rows // 3, n_rows)):
        for dim in (20, 250):
            d, lines = degs[rb:re], (dim + 31) // 32
            uses = np.sort(np.bincount(col[rowptr[rb]:rowptr[re]], minlength=n_cols))[::-1]
            miss = {v: 1 - uses[:32768 // v].sum() / uses.sum() for v in (1, 2, 4, 8)}
            E, slices = float(d.sum()), {v: -(-lines // v) for v in (1, 2, 4)}
            cost = {v: np.hypot(2.4 * E * lines * miss[v], E * lines + n * (0.2 * E + 2.5 * d.size) + 0.4 * (n * v - lines) * E)
                    + 2e4 * max(0.0, np.log2(1.2e6 / ((E + 8 * d.size) * n))) for v, n in slices.items()}
            best = min(cost, key=lambda v: (round(cost[v], 3), v))
            long = d[d >= 64]
            dense = 0.0 if transposed or (d >= max(n_cols // 20, 64)).sum() < 256 else d[d >= max(n_cols // 20, 64)].sum()
            old = -(0.26 * lines + 0.41) * d.sum() if transposed else -(0.5 * lines + 0.25) * d.sum() - 2.7 * lines * d.size
            gain = max(
                long.sum() * lines * miss[best] - 7 * long.size * lines * min(max(n_cols // 12288, 1), 8) - 0.15 * d.sum() - 1e6,
                0.56 * max(lines - 1.5, 0) * dense + long.sum() * lines * miss[8] + old - 1e6)
            got = B.adaqp_spmm_pieces_rule(rowptr, col, rb, re, n_cols, dim, transposed)
            assert got[0] == (0 if transposed and 1e5 <= E < 6 * d.size and lines >= 7 else best) and got[1] == pytest.approx(gain, rel=1e-9)
    col[rowptr[1]: rowptr[2]] = -1                                     # nothing to tile, lines all the same
    assert B.adaqp_spmm_pieces_rule(rowptr, col, 0, 2, n_cols, 20, transposed)[0] in (1, 2, 4)


@pytest.mark.parametrize("column", [149, 10_000, -1])
def test_spmm_pieces_rule_of_unsorted_rows(column):
    """Pieces take columns in any order: lines are told for rows that segments are refused for."""
    rowptr = np.array([0, 200, 400], np.int64)
    col = np.tile(np.arange(200, dtype=np.int32), 2)
    col[350] = column                                                  # twice, outside
    with pytest.raises(B.AdaqpError):
        B.adaqp_spmm_pieces_rule(rowptr, col, 0, 2, 10_000, 64)
    assert B.adaqp_spmm_pieces_rule(rowptr, col, 0, 2, 10_000, 64, segments=False)[0] in (1, 2, 4)
    assert B.adaqp_spmm_pieces_rule(rowptr[:2], col, 0, 1, 10_000, 64)[0] == B.adaqp_spmm_pieces_rule(rowptr[:2], col, 0, 1, 10_000, 64, segments=False)[0]


@pytest.mark.parametrize("lengths", [[], [1], [0, 5, 0], [256], [257], [768], [769], [5_000], [1] * 200, [700, 30, 40, 100, 2_000, 3] * 9,
                                     [700, 30, 900_000, 100, 5_000, 3] * 3])
@pytest.mark.parametrize("dim,lines", [(32, 1), (602, 2), (602, 4)])
def test_plan_spmm_pieces(lengths, dim, lines):
    """Pieces are consecutive, within their limits, and end with a segment or inside one; every part of a row goes to a place of its own."""
    lengths = np.array(lengths, np.int64)
    n_seg, S = lengths.size, B.SPMM_SEGMENTS
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    of_row = np.full((n_seg + 3, S), -1, np.int32)                     # rows of one, two and no segments, and one that is not of the plan
    row, seg = 1, 0
    while seg < n_seg:
        of_row[row, 2] = seg
        if seg % 3 == 1 and seg + 1 < n_seg:
            of_row[row, 7] = seg + 1
            seg += 1
        row, seg = row + 1, seg + 1
    of_row[-1, 0] = -2
    plan = B.adaqp_plan_spmm_pieces(ptr, of_row, dim, lines)
    pieces, dest = plan["pieces"], plan["dest"]
    assert pieces[0].tolist() == (0, 0, -1) and pieces[-1].tolist() == (ptr[-1], n_seg, -1)
    parts = [[] for _ in range(n_seg)]                                 # places that the parts of a segment go to
    for k, (here, there) in enumerate(zip(pieces[:-1], pieces[1:]), 1):
        assert 0 <= there["entry"] - here["entry"] <= plan["entries"] and 0 <= there["segment"] - here["segment"] <= 62
        for s in range(here["segment"], there["segment"]):
            parts[s].append(int(dest[s]))
        if there["partial"] == -1:
            assert there["entry"] == ptr[there["segment"]]
            continue
        assert max(here["entry"], ptr[there["segment"]]) < there["entry"] < ptr[there["segment"] + 1]
        if there["partial"] >= 0:
            parts[there["segment"]].append(int(there["partial"]))
        else:                                                          # handed to the next wave of the workgroup
            assert there["partial"] == -2 and plan["waves"] == 8 and k % 8 != 0
            assert np.all(pieces["partial"][1:][(pieces["segment"][1:] == there["segment"]) & (pieces["entry"][1:] > ptr[there["segment"]])] == -2)
    sums = dict(zip(plan["sum_row"].tolist(), zip(plan["sum_ptr"][:-1].tolist(), plan["sum_ptr"][1:].tolist())))
    assert plan["sum_ptr"][0] == 0 and np.all(np.diff(plan["sum_row"]) > 0) and of_row.shape[0] - 1 not in sums
    for r in range(of_row.shape[0] - 1):
        want = [p for s in of_row[r][of_row[r] >= 0] for p in parts[s]]
        assert want == ([-1 - r] if r not in sums else list(range(*sums[r])))
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_pieces(ptr, of_row, dim, 3)
    if n_seg:
        of_row[0, 0] = 0                                               # a segment of two rows
        with pytest.raises(B.AdaqpError):
            B.adaqp_plan_spmm_pieces(ptr, of_row, dim, lines)


@pytest.mark.parametrize("n_rows,n_cols,mean,transposed", [(0, 8, 0, False), (300, 50, 30, False), (3_000, 9_000, 90, False),
                                                           (3_000, 9_000, 90, True), (400, 5_000, 700, False)])
def test_spmm_segments_gain(n_rows, n_cols, mean, transposed):
    """The stated sum of savings and costs; rows that the plan would refuse have no segments and are refused where they were."""
    rng = np.random.default_rng(mean)
    degs = np.minimum((rng.pareto(1.2, size=n_rows) * mean / 3).astype(np.int64), n_cols)
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n_cols, size=d, replace=False)) for d in degs] or [[]]).astype(np.int32)
    for rb, re in ((0, n_rows), (n_rows // 3, n_rows)):
        got = B.adaqp_spmm_segments_gain(rowptr, col, rb, re, n_cols, 250, transposed)
        d, lines = degs[rb:re], 8
        dense = d[d >= max(n_cols // 20, 64)]
        want = -(0.26 * lines + 0.41) * d.sum() if transposed else \
            0.56 * (lines - 1.5) * (dense.sum() if dense.size >= 256 else 0) - (0.5 * lines + 0.25) * d.sum() - 2.7 * lines * d.size
        uses = np.sort(np.bincount(col[rowptr[rb]:rowptr[re]], minlength=n_cols))[::-1]
        best = want + d[d >= 64].sum() * lines
        if best > 0 or B.adaqp_spmm_tiled_pays(re - rb, int(d.sum())):
            want += d[d >= 64].sum() * lines * (1 - uses[:4096].sum() / max(uses.sum(), 1))
        assert got == pytest.approx(want, rel=1e-9, abs=1e-6)


def test_spmm_segments_gain_of_unsorted_rows():
    rowptr = np.array([0, 100, 200], np.int64)
    col = np.tile(np.arange(100, dtype=np.int32) * 100, 2)
    col[150] = col[149]                                                # a column twice
    assert B.adaqp_spmm_segments_gain(rowptr, col, 0, 1, 10_000, 64, True) > -np.inf
    assert B.adaqp_spmm_segments_gain(rowptr, col, 0, 2, 10_000, 64, True) == -np.inf
    col = np.tile(np.arange(200, dtype=np.int32), 2)
    col[250] = 10_000                                                  # outside; 200 entries per row: refused as ever
    with pytest.raises(B.AdaqpError):
        B.adaqp_spmm_segments_gain(np.array([0, 200, 400], np.int64), col, 0, 2, 10_000, 64, True)


def test_ranges_of_unsorted_rows_are_not_tiled():
    """A range that cannot gain is looked at too: it would be tiled with the range beside it, and the plan refuses such rows."""
    from types import SimpleNamespace
    import torch
    from paper_2306_01381_amd.layer import LayerStep
    rng = np.random.default_rng(5)
    n, short, n_cols = 12_000, 500, 60_000
    long_rows = np.sort(np.stack([rng.choice(n_cols, 110, replace=False) for _ in range(n)]), axis=1)
    col = np.concatenate([long_rows.reshape(-1), np.tile([9, 3, 5], short)]).astype(np.int32)
    rowptr = np.concatenate([np.arange(n) * 110, n * 110 + np.arange(short + 1) * 3]).astype(np.int64)
    assert B.adaqp_spmm_segments_gain(rowptr, col, 0, n, n_cols, 256) > B.SPMM_SEGMENTS_MIN_GAIN
    assert B.adaqp_spmm_segments_gain(rowptr, col, n, n + short, n_cols, 256) == -np.inf
    step = SimpleNamespace(p=SimpleNamespace(rowptr=rowptr, col=col, feat=np.empty((n_cols, 1))), feat=torch.zeros(1, 288), dim=256,
                           backward=False)
    assert LayerStep._ranges_to_tile(step, None, (0, n), (n, n + short)) == (True, False)
    assert LayerStep._ranges_to_tile(step, None, (n, n + short), (0, n), (n, n)) == (False, True, False)
    with pytest.raises(B.AdaqpError):                                  # an offset below zero
        B.adaqp_spmm_segments_gain(np.array([-5, 2], np.int64), col, 0, 1, n_cols, 256)


def test_spmm_planners_without_room():
    """Scratch per column that cannot be had is an error code or no gain, and no exception leaves the library."""
    code = """
import resource, numpy as np
from paper_2306_01381_amd import binding as B
rowptr, col, n_cols = np.array([0, 300], np.int64), np.arange(300, dtype=np.int32), 2**31 - 1
B.adaqp_plan_spmm_blocks(rowptr, col, 0, 1, 300, 64, 1)
limit = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize() + (256 << 20)
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
assert B.adaqp_spmm_segments_gain(rowptr, col, 0, 1, n_cols, 64) == -np.inf
for plan in (lambda: B.adaqp_plan_spmm_blocks(rowptr, col, 0, 1, n_cols, 64, 1), lambda: B.adaqp_plan_spmm_tiles(rowptr, col, 0, 1, n_cols)):
    try:
        plan()
    except B.AdaqpError as e:
        print("refused", e)
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert done.returncode == 0 and done.stdout.count("refused") == done.stdout.count("too small") == 2, (done.stdout, done.stderr[-2000:])


@pytest.mark.parametrize("n_rows,n_cols,min_len", [(1, 1, 1), (40, 33, 5), (130, 900, 60), (300, 2_000, 40)])
def test_plan_spmm_blocks(n_rows, n_cols, min_len):
    """A block lists exactly the distinct columns of its rows, each in its interval, ascending, steps filled with the last one."""
    rng = np.random.default_rng(n_rows)
    degs = np.minimum(rng.integers(0, n_cols + 1, size=n_rows) // rng.integers(1, 20, size=n_rows), n_cols)
    degs[0] = n_cols
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n_cols, size=d, replace=False)) for d in degs]).astype(np.int32)
    for rb, re in ((0, n_rows), (n_rows // 2, n_rows)):
        _, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        before = off.copy()
        plan = B.adaqp_plan_spmm_blocks(rowptr, col, rb, re, n_cols, 300, min_len, off)
        rows = [r for r in range(rb, re) if degs[r] >= min_len]
        if not rows:
            assert plan is None and np.array_equal(off, before)
            continue
        rows.sort(key=lambda r: (-degs[r], r))
        assert plan["rows"][:len(rows)].tolist() == rows and np.all(plan["rows"][len(rows):] == -1)
        assert plan["rows"].size == plan["n_blocks"] * B.SPMM_BLOCK_ROWS == -(-len(rows) // 128) * 128
        assert plan["n_pieces"] % 8 == 0 and plan["step_ptr"][-1] == plan["n_steps"] and np.all(np.diff(plan["step_ptr"]) >= 0)
        for b in range(plan["n_blocks"]):
            mine = [r for r in plan["rows"][b * 128: b * 128 + 128] if r >= 0]
            want = np.unique(np.concatenate([col[rowptr[r]: rowptr[r + 1]] for r in mine]))
            got = []
            for p in range(plan["n_pieces"]):
                s0, s1 = plan["step_ptr"][b * plan["n_pieces"] + p], plan["step_ptr"][b * plan["n_pieces"] + p + 1]
                c = plan["cols"][s0:s1].reshape(-1)
                lo = plan["col_begin"] + p * plan["piece_width"]
                assert np.all((c >= lo) & (c < lo + plan["piece_width"])) and np.all(np.diff(c) >= 0)
                distinct = np.unique(c)
                assert s1 - s0 == -(-distinct.size // 32) and np.array_equal(c[:distinct.size], distinct)
                got.append(distinct)
            assert np.array_equal(np.concatenate(got), want)
        taken = np.zeros(re - rb, dtype=bool)
        taken[np.array(rows) - rb] = True
        assert np.all(off[taken] == -1) and np.array_equal(off[~taken], before[~taken])
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_blocks(rowptr, col, 0, n_rows, n_cols, 300, 0)                                     # min_row_len < 1
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_blocks(np.array([0, 2], np.int64), np.array([5, 5], np.int32), 0, 1, 8, 300, 1)    # repeated column


def test_rule_that_decides_whether_a_panel_plan_pays():
    # one wave per (piece, 128-column chunk); fewer than ADAQP_SPMM_PANEL_MIN_WAVES of them do not fill the GPU
    assert not B.adaqp_spmm_panels_pay(0, 602) and not B.adaqp_spmm_panels_pay(100, 0)
    assert not B.adaqp_spmm_panels_pay(60, 602)            # one panel of a 602-column graph: 300 waves
    assert B.adaqp_spmm_panels_pay(1150, 602)              # eighteen panels: 5750 waves
    assert B.adaqp_spmm_panels_pay(2048, 128) and not B.adaqp_spmm_panels_pay(2047, 128)
    assert B.adaqp_spmm_panels_pay(410, 602) and not B.adaqp_spmm_panels_pay(409, 602)      # 5 chunks per piece
    # the planner binding turns a sized plan down on request and then leaves the tile table alone
    rng = np.random.default_rng(4)
    n_rows, n_cols = 40, 300
    degs = np.full(n_rows, 5)
    degs[:3] = 200
    rowptr = np.zeros(n_rows + 1, dtype=np.int64)
    np.cumsum(degs, out=rowptr[1:])
    col = np.concatenate([np.sort(rng.choice(n_cols, size=d, replace=False)) for d in degs]).astype(np.int32)
    val = rng.standard_normal(col.shape[0]).astype(np.float32)
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
    before = off.copy()
    assert B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, off, 100, 64,
                                    only_if_pays_for_dim=128) is None
    assert np.array_equal(off, before)
    assert B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, off, 100, 64) is not None
    assert not np.array_equal(off, before)


@pytest.mark.parametrize("n_cols,share,rows,dim,saves", [
    (24_000, 0.055, 1792, 64, False), (24_000, 0.055, 1792, 256, False), (24_000, 0.12, 256, 128, False), (24_000, 0.12, 256, 256, True),
    (24_000, 0.25, 512, 64, True), (24_000, 0.25, 256, 602, True), (90_000, 0.055, 1152, 256, False), (90_000, 0.12, 384, 64, False),
    (90_000, 0.12, 384, 96, True), (90_000, 0.12, 384, 602, True), (90_000, 0.12, 130, 32, False)])
def test_rule_that_decides_whether_blocks_save(n_cols, share, rows, dim, saves):
    """Timed with and without blocks: the faster way, where they differ."""
    steps = -(-rows // 128) * -(-n_cols // 32)
    assert bool(B.lib().adaqp_spmm_blocks_save(int(rows * share * n_cols), steps, dim, 0)) == saves


@pytest.mark.parametrize("entries,steps,dim,saves", [
    (294_861, 1_120, 32, False), (774_930, 926, 602, True), (2_315_452, 7_209, 64, False), (1_462_590, 3_833, 32, False),
    (1_462_590, 3_785, 400, True), (1_057_932, 3_234, 400, True), (2_839_519, 3_468, 64, True)])
def test_rule_that_decides_whether_blocks_save_beside_another_range(entries, steps, dim, saves):
    """Forward steps timed with and without blocks."""
    assert bool(B.lib().adaqp_spmm_blocks_save(entries, steps, dim, 1)) == saves


def test_plan_spmm_blocks_takes_the_rows_that_pay():
    """300 rows that list a quarter of the columns beside 8 000 that list a twentieth: all of them would be slower in blocks, the long
    ones are faster, and with few columns of H none are."""
    rng = np.random.default_rng(3)
    n_cols = 4_000
    degs = np.concatenate([np.full(8_000, 204), np.full(300, 1_000)])
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(n_cols, d, replace=False)) for d in degs]).astype(np.int32)
    n = degs.size
    _, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n, n_cols)
    before = off.copy()
    assert B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, 64, 200, off, only_if_pays_for_ld=64) is None
    assert np.array_equal(off, before)
    plan = B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, 602, 200, off, only_if_pays_for_ld=608)
    assert plan["n_rows_taken"] == 300 and np.array_equal(np.sort(plan["rows"][:300]), np.arange(8_000, n))
    assert np.all(off[8_000:] == -1) and np.array_equal(off[:8_000], before[:8_000])
    # where the caller has asked for tiles (the long rows: all of them would take a table of 133 MB), and where for blocks
    assert B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, 64, 200, only_if_pays_for_ld=64, if_slower=True)["n_rows_taken"] == 300
    assert B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, 64, 200)["n_rows_taken"] == n


def test_plan_spmm_blocks_bounds_its_table():
    """Rows at the threshold take ten times their bytes: no more than four times those of the range, or 64 MB."""
    assert B.lib().adaqp_spmm_blocks_most_steps(0) == B.lib().adaqp_spmm_blocks_most_steps(-1) == 4096
    assert B.lib().adaqp_spmm_blocks_most_steps(512 * 5_000) == 5_000
    n_cols, dim, n, d = 40_000, 602, 1_500, 3_000                      # 12 blocks x 1 250 steps: 246 MB; 4.5 M entries: 36 MB
    rng = np.random.default_rng(7)
    col = np.sort((np.arange(d) * 13 + rng.integers(0, n_cols, size=(n, 1))) % n_cols, axis=1).astype(np.int32)
    col[:300] = np.arange(37_000, n_cols)                              # rows that share their columns: few steps
    rowptr = np.arange(n + 1, dtype=np.int64) * d
    plan = B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, dim, 2_000)
    assert plan["n_steps"] > 4_500_000 // 512 and B.lib().adaqp_spmm_blocks_save(4_500_000, plan["n_steps"], dim, 0)
    for if_slower in (False, True):
        assert B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n_cols, dim, 2_000, only_if_pays_for_ld=608, if_slower=if_slower) is None
    small = B.adaqp_plan_spmm_blocks(rowptr, col, 0, 300, n_cols, dim, 2_000, only_if_pays_for_ld=608)
    assert small["n_rows_taken"] == 300 and small["n_steps"] <= 400


def test_version_says_how_the_structs_are_laid_out():
    """Whoever changes a layout gives it a version of its own."""
    sizes = {200: (152, 88, 1200)}
    assert (ctypes.sizeof(B.SpmmSegments), ctypes.sizeof(B.SpmmPieces), int(B.lib().adaqp_layer_desc_bytes())) == sizes[B.adaqp_version()]
    with open(os.path.join(ROOT, "include", "adaqp.h")) as f:
        assert f"#define ADAQP_VERSION {B.adaqp_version()}\n" in f.read()


def test_layer_desc_mirror_matches_the_library():
    import ctypes
    assert int(B.lib().adaqp_layer_desc_bytes()) == ctypes.sizeof(B.LayerDesc)
