"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Bars: packed bytes, (Z, S) and de-quantised fp32 values bit-exact; aggregation within
1e-5 * sum|terms| per output element (the fp64 oracle also returns that sum).
"""
import ctypes
import sys
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2306_01381_amd import binding as B                      # noqa: E402
from paper_2306_01381_amd.layer import LayerStep, SendPlan          # noqa: E402
from paper_2306_01381_amd.synth import CONFIGS, make_partition      # noqa: E402

DEV = "cuda:0"
SPMM_RTOL = 1e-5


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def _gpu_quantize(feat_np, dim, send_idx, bits, off, seed, packed_bytes, fill=0xAB):
    feat = torch.from_numpy(feat_np).to(DEV)
    packed = torch.full((max(packed_bytes, 4),), fill, dtype=torch.uint8, device=DEV)
    params = torch.full((max(len(send_idx), 1), 2), float("nan"), dtype=torch.float32, device=DEV)
    B.adaqp_quantize_pack(feat, dim, torch.from_numpy(send_idx).to(DEV), torch.from_numpy(bits).to(DEV),
                          torch.from_numpy(off).to(DEV), seed, packed, params)
    torch.cuda.synchronize()
    return packed.cpu().numpy(), params.cpu().numpy()


def _padded_cols(dim, ld):
    """Columns a line-padded output row gets zero-filled (torch allocations are at least 256-byte aligned)."""
    return min(ld, (dim + 31) // 32 * 32) if ld % 32 == 0 else dim


def _codec_case(oracle, feat_np, dim, send_idx, bits, peer, n_peers, seed, halo_rows=None, use_order=False):
    """Quantise on both sides, compare bytes and params; de-quantise on both sides, compare floats."""
    perm, off, pbp = oracle.plan_layout(dim, bits, peer, n_peers)
    perm_g, off_g, pbp_g = B.adaqp_plan_layout(dim, bits, peer, n_peers)
    assert np.array_equal(perm, perm_g) and np.array_equal(off, off_g) and np.array_equal(pbp, pbp_g)
    s_idx = np.ascontiguousarray(send_idx[perm], dtype=np.int32)
    s_bits = np.ascontiguousarray(bits[perm], dtype=np.uint8)
    nbytes = int(pbp[-1])
    want_packed, want_params, _ = oracle.quantize_pack(feat_np, dim, s_idx, s_bits, off, seed, nbytes)
    got_packed, got_params = _gpu_quantize(feat_np, dim, s_idx, s_bits, off, seed, nbytes)
    n = len(s_idx)
    assert np.array_equal(got_params[:n].view(np.uint32), want_params.view(np.uint32)), "(Z, S) differ"
    if nbytes:
        bad = np.nonzero(got_packed[:nbytes] != want_packed)[0]
        assert bad.size == 0, f"{bad.size} packed bytes differ, first at {bad[:5]}"
    # receive side, into a copy with a sentinel so that stray writes show
    ld = feat_np.shape[1]
    n_rows = feat_np.shape[0]
    halo = np.ascontiguousarray(halo_rows if halo_rows is not None
                                else np.random.default_rng(seed).permutation(n_rows)[:n], dtype=np.int32)
    want = np.full((n_rows, ld), np.float32(-123.5))
    oracle.unpack_dequant(want_packed, want_params, s_bits, off, halo, dim, want)
    want[halo, dim:_padded_cols(dim, ld)] = 0.0            # whole-line writes zero the row padding
    got = torch.full((n_rows, ld), -123.5, dtype=torch.float32, device=DEV)
    order = torch.from_numpy(B.adaqp_plan_recv_order(halo)).to(DEV) if use_order else None
    B.adaqp_unpack_dequant(torch.from_numpy(want_packed if nbytes else np.zeros(4, np.uint8)).to(DEV),
                           torch.from_numpy(want_params if n else np.zeros((1, 2), np.float32)).to(DEV),
                           torch.from_numpy(s_bits).to(DEV), torch.from_numpy(off).to(DEV),
                           torch.from_numpy(halo).to(DEV), dim, got, order=order)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32)), "de-quantised rows differ"


@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 602), (256, 256), (300, 300), (300, 301), (7, 7), (1, 1),
                                    (8, 12), (9, 9), (33, 40), (63, 63), (64, 64), (65, 66), (1000, 1000),
                                    (4096, 4096), (4100, 4100), (5000, 5001),
                                    # line-padded pitches: whole-line reads and writes, ragged last vector
                                    (602, 608), (300, 320), (7, 32), (33, 64), (1, 32), (130, 160), (1000, 1024),
                                    (250, 256), (2047, 2048), (2049, 2080), (4100, 4128), (602, 640), (602, 604)])
def test_codec_shapes(oracle, dim, ld):
    _say(f"codec dim={dim} ld={ld}")
    rng = np.random.default_rng(dim * 7 + ld)
    n_rows, n = 300, 211                       # several blocks of rows and a ragged last block
    feat = rng.standard_normal((n_rows, ld), dtype=np.float32)
    feat[:, dim:] = np.float32(1e30)           # padding must never enter min / max
    feat[3] = 1.25                                                    # constant row
    feat[4, : dim // 2] = 0.0
    feat[5] = np.maximum(feat[5], 0)
    feat[6] *= np.float32(1e-3)
    send = rng.integers(0, n_rows, size=n).astype(np.int32)
    send[:8] = np.arange(8)
    bits = rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=n)
    peer = np.sort(rng.integers(0, 3, size=n)).astype(np.int32)
    _codec_case(oracle, feat, dim, send, bits, peer, 3, seed=dim, use_order=(dim % 2 == 0))


@pytest.mark.parametrize("b", [2, 4, 8])
def test_codec_single_width_and_seeds(oracle, b):
    _say(f"codec single width b={b}")
    rng = np.random.default_rng(b)
    feat = rng.standard_normal((64, 602), dtype=np.float32)
    for seed in (0, 1, 2**32 + 5, 2**64 - 1):
        _codec_case(oracle, feat, 602, np.arange(64, dtype=np.int32), np.full(64, b, np.uint8),
                    np.zeros(64, np.int32), 1, seed)


@pytest.mark.parametrize("dim,ld", [(24, 24), (602, 608), (300, 320), (5000, 5000)])
def test_codec_tiny_ranges_and_signed_zeros(oracle, dim, ld):
    """Rows at the bottom of fp32 (ranges from 1e-30 down to the smallest denormal: the scale with the 2^16 folded
    in overflows, then the reciprocal itself), rows whose minimum is reached by both -0.0 and +0.0, constant rows
    of either zero - next to ordinary rows in the same waves, every width."""
    _say(f"codec tiny ranges dim={dim} ld={ld}")
    rng = np.random.default_rng(dim)
    scales = [1.0, 1e-30, 1e-33, 1e-36, 3e-38, 1e-39, 1e-42, 3e-45, 1e-3]
    n_rows = 6 * len(scales)
    feat = np.zeros((n_rows, ld), dtype=np.float32)
    for i, sc in enumerate(scales):
        u = rng.random((6, dim))
        u[:, 0], u[:, -1] = 0.0, 1.0
        base = np.array([0.0, sc * 8, -sc * 3, 1e-20, 0.0, 0.0])[:, None]
        rows = (base + u * sc).astype(np.float32)
        rows[4] = np.float32(sc)
        rows[5, 1:] = rows[5, 0]
        if dim > 1:
            rows[5, 1] = np.nextafter(rows[5, 0], np.float32(1), dtype=np.float32)
        feat[6 * i: 6 * i + 6, :dim] = rows
    zeros = np.zeros((6, ld), dtype=np.float32)
    zeros[0, :dim] = np.maximum(rng.standard_normal(dim), 0)      # ReLU-like row: minimum +0.0 ...
    zeros[0, dim // 2] = -0.0                                      # ... and -0.0
    zeros[0, 0] = 0.0
    zeros[1, :dim] = -np.maximum(rng.standard_normal(dim), 0)     # maximum reached by both zeros
    zeros[1, 0] = 0.0
    zeros[1, dim - 1] = -0.0
    zeros[2, :dim] = -0.0                                          # constant -0.0
    zeros[3, :dim] = 0.0
    zeros[3, dim - 1] = -0.0                                       # "constant" row holding both zeros
    zeros[4, :dim] = rng.standard_normal(dim).astype(np.float32)
    zeros[5, :dim] = np.where(rng.random(dim) < 0.5, 0.0, -0.0)   # a mixture of the two zeros only
    feat = np.concatenate([feat, zeros], 0)
    n_rows = feat.shape[0]                                         # the rows that are sent
    feat = np.concatenate([feat, rng.standard_normal((2 * n_rows, ld), dtype=np.float32)], 0)   # room to receive
    feat[:, dim:] = np.float32(1e30)
    for b in (2, 4, 8):
        send = np.concatenate([np.arange(n_rows), rng.permutation(n_rows)]).astype(np.int32)
        bits = np.full(send.shape[0], b, np.uint8)
        _codec_case(oracle, feat, dim, send, bits, np.zeros(send.shape[0], np.int32), 1, seed=17 + b)
    send = np.tile(np.arange(n_rows), 3).astype(np.int32)
    bits = rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=send.shape[0])
    peer = np.sort(rng.integers(0, 2, size=send.shape[0])).astype(np.int32)
    _codec_case(oracle, feat, dim, send, bits, peer, 2, seed=99)


def test_codec_c0(oracle):
    _say("codec c0")
    p = make_partition(CONFIGS["c0"])
    _codec_case(oracle, p.feat, p.cfg.dim, p.send_idx, p.bits, p.peer_of_slot, p.cfg.n_peers, seed=0,
                halo_rows=None)


def test_codec_distributions(oracle):
    """The value distributions of the four workloads at reduced row counts."""
    for name in ("c1", "c2", "c3", "c4"):
        _say(f"codec distribution {name}")
        cfg = replace(CONFIGS[name], n_local=3000, n_halo=2500, n_send=1500, mean_degree=6.0)
        p = make_partition(cfg)
        feat = p.feat if not cfg.backward else np.concatenate([p.feat, p.feat[:1600] * 3], 0)
        send = p.send_idx if not cfg.backward else (p.send_idx % feat.shape[0]).astype(np.int32)
        _codec_case(oracle, np.ascontiguousarray(feat), cfg.dim, send, p.bits, p.peer_of_slot, cfg.n_peers, seed=11)


def test_codec_skips_invalid_slots_and_empty_input(oracle):
    _say("codec invalid slots")
    rng = np.random.default_rng(0)
    dim = 40
    feat = rng.standard_normal((10, dim), dtype=np.float32)
    send = np.array([0, 99, 2, -1, 4], dtype=np.int32)              # 99 and -1 are out of range
    bits = np.array([2, 2, 3, 4, 8], dtype=np.uint8)                # 3 is not a width
    off = np.array([0, 12, 24, 48, 68], dtype=np.int64)
    nbytes = 68 + 40
    got_packed, got_params = _gpu_quantize(feat, dim, send, bits, off, 1, nbytes, fill=0xCD)
    # the oracle rejects invalid slots outright and keys the random stream by position: give it valid
    # stand-ins at the skipped positions and compare only the bytes of the valid slots
    send_v, bits_v = send.copy(), bits.copy()
    send_v[[1, 3]] = 0
    bits_v[2] = 4
    full_packed, full_params, _ = oracle.quantize_pack(feat, dim, send_v, bits_v, off, 1, nbytes)
    assert np.array_equal(got_packed[0:12], full_packed[0:12])
    assert np.array_equal(got_packed[68:108], full_packed[68:108])
    assert np.all(got_packed[12:68] == 0xCD)                          # skipped slots wrote nothing
    assert np.array_equal(got_params[[0, 4]].view(np.uint32), full_params[[0, 4]].view(np.uint32))
    assert np.isnan(got_params[[1, 2, 3]]).all()
    # a row that would overrun the buffer is skipped too
    got_packed, got_params = _gpu_quantize(feat, dim, send[:1], np.array([8], np.uint8), np.array([80], np.int64),
                                           1, 100, fill=0xCD)
    assert np.all(got_packed == 0xCD) and np.isnan(got_params[0]).all()
    # empty input
    e32, e8, e64 = np.zeros(0, np.int32), np.zeros(0, np.uint8), np.zeros(0, np.int64)
    got_packed, _ = _gpu_quantize(feat, dim, e32, e8, e64, 1, 0, fill=0xCD)
    assert np.all(got_packed == 0xCD)


# ------------------------------------------------------------------------------------------------------
# trace for the bit-width assigner (beta of Sec. 4.2)
# ------------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (602, 602), (300, 320), (7, 7), (5000, 5000)])
def test_quantize_trace_beta(oracle, dim, ld):
    _say(f"beta trace dim={dim} ld={ld}")
    rng = np.random.default_rng(dim)
    n_rows, n = 120, 97
    feat = rng.standard_normal((n_rows, ld), dtype=np.float32) * rng.choice([1e-3, 1.0, 50.0], size=(n_rows, 1)).astype(np.float32)
    feat[2, :dim] = 0.75
    feat[:, dim:] = np.float32(1e30)
    send = rng.integers(0, n_rows, size=n).astype(np.int32)
    send[0] = 2
    bits = np.sort(rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=n))
    perm, off, pbp = oracle.plan_layout(dim, bits, np.zeros(n, np.int32), 1)
    alpha_sq = rng.uniform(0.01, 3.0, size=n).astype(np.float32)
    want_packed, want_params, _ = oracle.quantize_pack(feat, dim, send, bits, off, 9, int(pbp[-1]))
    want_beta = oracle.trace_beta(feat, dim, send, alpha_sq)
    packed = torch.zeros(int(pbp[-1]), dtype=torch.uint8, device=DEV)
    params = torch.zeros((n, 2), dtype=torch.float32, device=DEV)
    beta = torch.full((n,), float("nan"), dtype=torch.float32, device=DEV)
    B.adaqp_quantize_pack_trace(torch.from_numpy(feat).to(DEV), dim, torch.from_numpy(send).to(DEV),
                                torch.from_numpy(bits).to(DEV), torch.from_numpy(off).to(DEV), 9, packed, params,
                                torch.from_numpy(alpha_sq).to(DEV), beta)
    torch.cuda.synchronize()
    assert np.array_equal(packed.cpu().numpy(), want_packed)
    assert np.array_equal(params.cpu().numpy().view(np.uint32), want_params.view(np.uint32))
    assert np.array_equal(beta.cpu().numpy().view(np.uint32), want_beta.view(np.uint32))
    assert want_beta[0] == 0.0
    with pytest.raises(B.AdaqpError):
        B.lib()            # keeps the import used
        B._check(B.lib().adaqp_quantize_pack_trace(1, 1, 8, 8, 1, 1, 1, 1, 0, 1, 8, 1, None, 1, None), "one NULL")


# ------------------------------------------------------------------------------------------------------
# backward receive: de-quantise and add
# ------------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (602, 602), (256, 256), (300, 320), (7, 7), (1, 1),
                                    (33, 40), (1100, 1120), (2500, 2500)])
def test_dequant_add(oracle, dim, ld):
    _say(f"dequant add dim={dim} ld={ld}")
    rng = np.random.default_rng(dim + ld)
    n_rows, n = 180, 400
    src = rng.standard_normal((n, dim), dtype=np.float32) * np.float32(1e-3)
    bits = rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=n)
    peer = np.sort(rng.integers(0, 7, size=n)).astype(np.int32)
    perm, off, pbp = oracle.plan_layout(dim, bits, peer, 7)
    s_bits = np.ascontiguousarray(bits[perm])
    packed, params, _ = oracle.quantize_pack(src, dim, perm.astype(np.int32), s_bits, off, 5, int(pbp[-1]))
    dst = rng.integers(60, 160, size=n).astype(np.int32)          # ~4 messages per row, rows 0..59 untouched
    dst[:3] = [-1, n_rows, 61]                                      # two out-of-range destinations: skipped
    order, seg_ptr = B.adaqp_plan_recv_segments(dst)
    grad0 = rng.standard_normal((n_rows, ld), dtype=np.float32)
    want = grad0.copy()
    ok = (dst >= 0) & (dst < n_rows)
    idx = np.nonzero(ok)[0]
    oracle.unpack_dequant_add(packed, params[idx], s_bits[idx], off[idx], dst[idx], dim, want)
    got = torch.from_numpy(grad0).to(DEV)
    B.adaqp_unpack_dequant_add(torch.from_numpy(packed).to(DEV), torch.from_numpy(params).to(DEV),
                               torch.from_numpy(s_bits).to(DEV), torch.from_numpy(off).to(DEV),
                               torch.from_numpy(dst).to(DEV), torch.from_numpy(order).to(DEV),
                               torch.from_numpy(seg_ptr).to(DEV), dim, got)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))


# ------------------------------------------------------------------------------------------------------
# aggregation
# ------------------------------------------------------------------------------------------------------

def _gpu_spmm(rowptr, col, val, rb, re, H, dim, nnz_range=-1, out_fill=7.0, ldo=None):
    n_rows_total = rowptr.shape[0] - 1
    ldo = dim if ldo is None else ldo
    out = torch.full((n_rows_total, ldo), out_fill, dtype=torch.float32, device=DEV)
    nz = int(rowptr[re] - rowptr[rb]) if nnz_range == "exact" else -1
    ws_bytes = B.adaqp_spmm_workspace_bytes(re - rb, nz if nz >= 0 else len(col), dim)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    colt = torch.from_numpy(col).to(DEV) if len(col) else torch.zeros(1, dtype=torch.int32, device=DEV)[:0]
    valt = torch.from_numpy(val).to(DEV) if len(val) else torch.zeros(1, dtype=torch.float32, device=DEV)[:0]
    B.adaqp_spmm_csr(torch.from_numpy(rowptr).to(DEV), colt, valt, rb, re, torch.from_numpy(H).to(DEV), dim, out,
                     ws, nnz_range=nz)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check_spmm(oracle, rowptr, col, val, rb, re, H, dim, **kw):
    got = _gpu_spmm(rowptr, col, val, rb, re, H, dim, **kw)
    Hc = np.ascontiguousarray(H[:, :dim]) if H.shape[1] != dim else H
    want, mag = oracle.spmm_csr(rowptr, col, val, rb, re, Hc, dim)
    err = np.abs(got[rb:re, :dim].astype(np.float64) - want)
    tol = SPMM_RTOL * mag + 1e-30
    worst = float((err / tol).max()) if err.size else 0.0
    assert worst <= 1.0, f"worst error {worst:.3f} x tolerance"
    assert np.all(got[:rb] == 7.0) and np.all(got[re:] == 7.0), "rows outside the range were written"
    ldo, ldh = got.shape[1], H.shape[1]
    zero_to = _padded_cols(dim, ldo) if (ldo % 32 == 0 and ldh % 32 == 0) else dim
    assert np.all(got[rb:re, dim:zero_to] == 0.0), "row padding of written rows must be zero"
    assert np.all(got[:, zero_to:] == 7.0), "columns past the padded row were written"
    return got


def _random_graph(rng, n_rows, n_cols, degs):
    rowptr = np.zeros(n_rows + 1, dtype=np.int64)
    cols = []
    for r in range(n_rows):
        d = int(min(degs[r], n_cols))
        c = np.sort(rng.choice(n_cols, size=d, replace=False)) if d else np.zeros(0, np.int64)
        cols.append(c)
        rowptr[r + 1] = rowptr[r] + d
    col = np.concatenate(cols).astype(np.int32) if cols else np.zeros(0, np.int32)
    val = rng.standard_normal(col.shape[0]).astype(np.float32)
    return rowptr, col, val


@pytest.mark.parametrize("dim,ldh", [(128, 128), (602, 602), (256, 256), (300, 300), (1, 1), (7, 9), (66, 66),
                                     (130, 132), (2048, 2048), (2052, 2052), (515, 515),
                                     # line-padded pitches (H padding holds NaN: it must never reach the output)
                                     (602, 608), (300, 320), (7, 32), (250, 256), (2049, 2080), (129, 160)])
def test_spmm_shapes(oracle, dim, ldh):
    _say(f"spmm dim={dim} ldh={ldh}")
    rng = np.random.default_rng(dim)
    n_rows, n_cols = 700, 900
    degs = rng.integers(0, 12, size=n_rows)
    degs[10] = 800                                                     # a row far longer than one piece
    degs[11] = 0
    degs[500:520] = 0                                                  # a run of empty rows
    degs[699] = 300                                                    # heavy last row
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ldh), np.nan, dtype=np.float32)
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    ldo = ldh if ldh % 32 == 0 else dim
    _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=ldo)
    _check_spmm(oracle, rowptr, col, val, 9, 12, H, dim, nnz_range="exact", ldo=ldo)
    _check_spmm(oracle, rowptr, col, val, 495, 700, H, dim, nnz_range="exact", ldo=ldo)
    _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=dim + 3)            # unpadded output


@pytest.mark.parametrize("dim,n_cols", [(d, 700) for d in (32, 60, 96, 128, 160, 250, 288)] +  # four lines per slice: every
                         [(d, 50_000) for d in (32, 60, 96, 250)] + [(60, 201_000), (100, 201_000)])   # last width; one; two
def test_spmm_sliced_edges(oracle, dim, n_cols):
    """Line-padded layout: row ends at every place of a step, more row ends than a chunk takes, rows of a chunk's length
    and of many shares', empty rows at both ends; the launch sized for far fewer and far more entries than there are."""
    _say(f"spmm sliced dim={dim} n_cols={n_cols}")
    rng = np.random.default_rng(dim + n_cols)
    degs = np.concatenate([np.zeros(70), np.ones(130), np.arange(40), [383, 384, 385, 8, 16, 0, 0], np.full(60, 23),
                           [20_000, 5, 3_000], rng.integers(0, 90, size=3000), np.zeros(3)]).astype(int)
    rowptr, col, val = _random_graph(rng, degs.shape[0], n_cols, degs)
    assert len(col) > 110_000                               # fewer go along the merge path
    ld = _padded_cols(dim, 64 * dim)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    n_rows = degs.shape[0]
    _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=ld)
    _check_spmm(oracle, rowptr, col, val, 65, n_rows - 1, H, dim, nnz_range="exact", ldo=ld)
    _check_spmm(oracle, rowptr, col, val, 190, 300, H, dim, ldo=ld)
    out = torch.full((n_rows, ld), 7.0, device=DEV)
    ws = torch.empty(max(B.adaqp_spmm_workspace_bytes(n_rows, len(col), dim), 256), dtype=torch.uint8, device=DEV)
    B.adaqp_spmm_csr(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV), torch.from_numpy(val).to(DEV), 0,
                     n_rows, torch.from_numpy(H).to(DEV), dim, out, ws, nnz_range=100_000)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    assert np.all(np.abs(out.cpu().numpy()[:, :dim].astype(np.float64) - want) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("dim,ldh,ldo", [(4, 4, 4), (5, 7, 5), (31, 31, 33), (33, 33, 33), (97, 97, 98), (100, 100, 100),
                                         (128, 129, 128), (130, 160, 130), (131, 131, 160), (301, 301, 301),
                                         (515, 515, 515), (516, 517, 516), (517, 517, 517)])   # chunks end in 3, 4, 5 columns
def test_spmm_sliced_unpadded(oracle, dim, ldh, ldo):
    """Rows that start anywhere and share lines: the last columns of a row, nothing read or written beside it."""
    _say(f"spmm sliced unpadded dim={dim} ldh={ldh} ldo={ldo}")
    rng = np.random.default_rng(dim)
    degs = np.concatenate([np.zeros(70), np.arange(40), [383, 384, 385, 8, 16, 0, 0], np.full(60, 23), [700, 5, 600],
                           rng.integers(40, 160, size=1200), np.zeros(3)]).astype(int)
    n_rows, n_cols = degs.shape[0], 700
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    assert len(col) > 100_000 and len(col) // n_rows >= 64  # long rows and enough of them: the sliced kernel
    H = np.full((n_cols, ldh), np.nan, dtype=np.float32)    # what lies between the rows must never reach a sum
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=ldo)
    _check_spmm(oracle, rowptr, col, val, 65, n_rows - 1, H, dim, nnz_range="exact", ldo=ldo)


def test_spmm_degenerate(oracle):
    _say("spmm degenerate")
    rng = np.random.default_rng(1)
    H = rng.standard_normal((5, 16), dtype=np.float32)
    # all rows empty
    rowptr = np.zeros(41, dtype=np.int64)
    got = _check_spmm(oracle, rowptr, np.zeros(0, np.int32), np.zeros(0, np.float32), 0, 40, H, 16)
    assert np.all(got == 0)
    # a single row holding everything
    rowptr = np.array([0, 5], dtype=np.int64)
    _check_spmm(oracle, rowptr, np.arange(5, dtype=np.int32), np.ones(5, np.float32), 0, 1, H, 16)
    # one very long row between empty ones (more entries than any piece)
    n = 5000
    Hbig = rng.standard_normal((n, 64), dtype=np.float32)
    rowptr = np.array([0, 0, 0, n, n, n], dtype=np.int64)
    _check_spmm(oracle, rowptr, np.arange(n, dtype=np.int32), rng.standard_normal(n).astype(np.float32), 0, 5,
                Hbig, 64)
    # out-of-range columns are skipped, not read
    rowptr = np.array([0, 3], dtype=np.int64)
    col = np.array([0, 77, 2], dtype=np.int32)
    val = np.array([1.0, 5.0, 2.0], dtype=np.float32)
    got = _gpu_spmm(rowptr, col, val, 0, 1, H, 16)
    assert np.allclose(got[0], H[0] + 2 * H[2], rtol=1e-6)
    # empty range
    got = _gpu_spmm(np.array([0, 3], dtype=np.int64), col, val, 1, 1, H, 16)
    assert np.all(got == 7.0)


@pytest.mark.parametrize("dim,ldh", [(256, 288), (96, 96), (60, 61)])       # one line per slice, three, rows that share lines
@pytest.mark.parametrize("base", [0, 1, 31])                                # first entry of the range: chunks end at multiples of 32
def test_spmm_sliced_chunks(oracle, dim, ldh, base):
    """Rows that end next to the bounds of a chunk (768 entries) and of its parts (384): one to two entries off them, empty rows
    there, rows of several chunks, and runs of more than 63 row ends, which cut a chunk short."""
    _say(f"spmm sliced chunks dim={dim} ldh={ldh} base={base}")
    rng = np.random.default_rng(77)
    near = [384 + d for d in (-2, -1, 0, 0, 1, 2)] + [768 + d for d in (-1, 0, 1)] + [2304, 353, 31, 0, 0, 1, 736, 32, 383]
    degs = np.array([base] + (near + [0] * 70 + near[::-1] + [8] * 70 + [1] * 130) * 16)
    rowptr, col, val = _random_graph(rng, degs.size, 20_000, degs)
    H = np.zeros((20_000, ldh), dtype=np.float32)
    H[:, :dim] = rng.standard_normal((20_000, dim))
    assert rowptr[1] == base and rowptr[-1] >= 150_000
    _check_spmm(oracle, rowptr, col, val, 1, degs.size, H, dim)


@pytest.mark.parametrize("dim,n_cols", [(608, 64), (608, 12_000), (601, 64)])       # four lines per slice; one; rows that share lines
def test_spmm_sliced_long_sums(dim, n_cols):
    """Rows far longer than a wave's share of a launch with few shares (16 000 entries each): no addition chain is longer than
    a chunk's 48 steps per group, the chunks of a share (43) or the shares of a row (8), plus the three additions across
    the groups and one between chain and chain.  The term is one whose running sum always rounds the same way (2 000
    additions: 3e-5 off), so that the bound is what is measured."""
    _say(f"spmm sliced long sums dim={dim} n_cols={n_cols}")
    n_rows, degree, term = 66, 100_000, np.float32(1.9876709)
    rowptr = torch.arange(n_rows + 1, dtype=torch.int64, device=DEV) * degree
    col = torch.arange(n_rows * degree, dtype=torch.int32, device=DEV) % n_cols
    val = torch.ones(n_rows * degree, device=DEV)
    H = torch.full((n_cols, dim), float(term), device=DEV)
    out = torch.full((n_rows, dim), 7.0, device=DEV)
    ws = torch.empty(B.adaqp_spmm_workspace_bytes(n_rows, n_rows * degree, dim), dtype=torch.uint8, device=DEV)
    B.adaqp_spmm_csr(rowptr, col, val, 0, n_rows, H, dim, out, ws)
    torch.cuda.synchronize()
    error = float((out.double() / (degree * float(term)) - 1).abs().max())
    assert error <= (48 + 43 + 8 + 3 + 3) * 2.0 ** -24, error


@pytest.mark.parametrize("dim", [16, 33, 64, 300, 2080])
def test_spmm_no_columns(dim):
    """A matrix without rows, of every pitch: nothing is read of it, every row of out is zero."""
    _say(f"spmm no columns dim={dim}")
    for ld in (dim, (dim + 31) // 32 * 32, (dim + 31) // 32 * 32 + 32):
        out = torch.full((50, ld), 7.0, device=DEV)
        ws = torch.empty(max(B.adaqp_spmm_workspace_bytes(50, 0, dim), 256), dtype=torch.uint8, device=DEV)
        B.adaqp_spmm_csr(torch.zeros(51, dtype=torch.int64, device=DEV), torch.zeros(0, dtype=torch.int32, device=DEV),
                         torch.zeros(0, device=DEV), 0, 50, torch.zeros((0, ld), device=DEV), dim, out, ws)
        torch.cuda.synchronize()
        zero_to = _padded_cols(dim, ld)
        assert bool((out[:, :zero_to] == 0.0).all()) and bool((out[:, zero_to:] == 7.0).all())


def test_spmm_is_deterministic(oracle):
    _say("spmm determinism")
    p = make_partition(CONFIGS["c0"])
    a = _gpu_spmm(p.rowptr, p.col, p.val, 0, p.n_rows, p.feat, p.cfg.dim)
    b = _gpu_spmm(p.rowptr, p.col, p.val, 0, p.n_rows, p.feat, p.cfg.dim)
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_spmm_c0_and_nonnegative_long_rows(oracle):
    _say("spmm c0")
    p = make_partition(CONFIGS["c0"])
    _check_spmm(oracle, p.rowptr, p.col, p.val, 0, p.n_rows, p.feat, p.cfg.dim)
    _check_spmm(oracle, p.rowptr, p.col, p.val, 0, p.n_central, p.feat, p.cfg.dim, nnz_range="exact")
    _check_spmm(oracle, p.rowptr, p.col, p.val, p.n_central, p.n_rows, p.feat, p.cfg.dim, nnz_range="exact")
    # non-negative features and weights: partial sums grow monotonically, the hardest case for fp32 sums
    rng = np.random.default_rng(2)
    n_cols = 30000
    degs = np.array([25000, 3, 12000, 1])
    rowptr, col, val = _random_graph(rng, 4, n_cols, degs)
    val = np.abs(val)
    H = np.abs(rng.standard_normal((n_cols, 256), dtype=np.float32))
    _check_spmm(oracle, rowptr, col, val, 0, 4, H, 256)


# ------------------------------------------------------------------------------------------------------
# aggregation that reads received rows straight from the receive buffer
# ------------------------------------------------------------------------------------------------------

def _packed_case(oracle, rng, n_cols, n_halo, dim, ldh, seed):
    """Received rows for n_halo random columns: (halo, bits, off, packed, params, H_plain, H_ref) where H_plain
    holds NaN in the received rows and H_ref holds what the oracle de-quantises there."""
    halo = np.ascontiguousarray(rng.permutation(n_cols)[:n_halo], dtype=np.int32)
    bits = rng.choice(np.array([2, 4, 8], dtype=np.uint8), size=n_halo)
    peer = np.sort(rng.integers(0, 3, size=n_halo)).astype(np.int32)
    perm, off, pbp = oracle.plan_layout(dim, bits, peer, 3)
    bits = np.ascontiguousarray(bits[perm])
    halo = np.ascontiguousarray(halo[perm])
    src = (rng.standard_normal((n_halo, dim)) * rng.uniform(0.1, 3.0, size=(n_halo, 1))).astype(np.float32)
    packed, params, _ = oracle.quantize_pack(src, dim, np.arange(n_halo, dtype=np.int32), bits, off, seed, int(pbp[-1]))
    H_plain = np.full((n_cols, ldh), np.nan, dtype=np.float32)
    H_plain[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    H_ref = H_plain[:, :dim].copy()
    oracle.unpack_dequant(packed, params, bits, off, halo, dim, H_ref)
    H_plain[halo] = np.nan                                  # the fused path must never read these rows
    return halo, bits, off, packed, params, H_plain, H_ref


def _gpu_spmm_packed(rowptr, col, val, rb, re, H, dim, slot_of_row, packed, params, bits, off, ldo):
    out = torch.full((rowptr.shape[0] - 1, ldo), 7.0, dtype=torch.float32, device=DEV)
    ws = torch.empty(max(B.adaqp_spmm_workspace_bytes(re - rb, len(col), dim), 256), dtype=torch.uint8, device=DEV)
    B.adaqp_spmm_csr_packed(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV),
                            torch.from_numpy(val).to(DEV), rb, re, torch.from_numpy(H).to(DEV), dim, out,
                            torch.from_numpy(slot_of_row).to(DEV), torch.from_numpy(packed).to(DEV),
                            torch.from_numpy(params).to(DEV), torch.from_numpy(bits).to(DEV),
                            torch.from_numpy(off).to(DEV), ws)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("dim,n_rows", [(65, 9_000), (72, 17_000), (129, 17_000), (130, 9_000), (160, 17_000), (161, 9_000)])
def test_spmm_longer_pieces(oracle, dim, n_rows):
    """Rows that share lines, pieces of 64 and 128 steps and (161 columns) of 32: rows of every length around a chain's and a piece's, the
    same bits from packed rows."""
    _say(f"spmm longer pieces dim={dim} rows={n_rows}")
    rng = np.random.default_rng(7000 + dim)
    n_cols, ld = 3_000, dim if dim != 160 else 164
    degs = rng.integers(0, 48, size=n_rows)
    degs[:18] = [2_900, 0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 255, 256, 257]
    degs[400:700], degs[-1] = 0, 1_500
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    assert n_rows + len(col) > 6_000 * (32 if n_rows == 9_000 else 64) and len(col) > 110_000
    halo, bits, off, packed, params, H_plain, H_ref = _packed_case(oracle, rng, n_cols, 1_000, dim, ld, seed=5)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)
    H[:, :dim] = H_ref
    plain = _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=ld)
    fused = _gpu_spmm_packed(rowptr, col, val, 0, n_rows, H_plain, dim, B.adaqp_plan_slot_of_row(n_cols, halo), packed, params, bits, off, ld)
    assert np.array_equal(plain.view(np.uint32), fused.view(np.uint32))


@pytest.mark.parametrize("dim,ld", [(5, 5), (301, 301), (512, 513), (513, 513), (512, 514), (514, 514), (512, 512), (516, 516), (608, 608)])
def test_spmm_joined_pieces(oracle, dim, ld):
    """Pieces of 32 steps, four to a workgroup: rows that end with a piece and with a workgroup, that begin and end in any two of its waves, that
    fill several workgroups, empty ones between them; widths whose parts meet in LDS and (514, 516, 608 columns) leave a carry each."""
    _say(f"spmm joined pieces dim={dim} ld={ld}")
    rng = np.random.default_rng(9100 + dim + ld)
    n_cols = 1_500
    degs = np.concatenate([[31, 31, 63, 127, 126, 0, 0, 128, 1_400, 5, 30, 33, 700, 0, 1], rng.integers(0, 90, 200), [0] * 140, rng.integers(0, 6, 300),
                           [95, 32, 64, 1_023, 0, 0, 3, 129]])
    rowptr, col, val = _random_graph(rng, degs.size, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)
    H[:, :dim] = rng.standard_normal((n_cols, dim))
    for rb, re in ((0, degs.size), (8, 9), (3, degs.size - 2)):
        once = _check_spmm(oracle, rowptr, col, val, rb, re, H, dim, ldo=ld)
        assert np.array_equal(once.view(np.uint32), _gpu_spmm(rowptr, col, val, rb, re, H, dim, ldo=ld).view(np.uint32))


@pytest.mark.parametrize("dim,ld,n_rows,joined", [(33, 33, 2_000, False), (301, 301, 2_000, False), (300, 320, 2_000, False), (65, 65, 36_900, False),
                                                  (301, 301, 10_000, True), (512, 512, 6_000, True)])
def test_spmm_merge_path_of_short_rows(oracle, dim, ld, n_rows, joined):
    """Rows of two or three entries along the merge path: a carry per piece in small calls, joined pieces in larger ones; a row over several
    workgroups among them, the same bits from packed rows and in a second call."""
    _say(f"spmm short rows dim={dim} ld={ld} rows={n_rows}")
    rng = np.random.default_rng(8100 + dim + n_rows)
    n_cols = 3_000
    degs = rng.integers(0, 6, size=n_rows)
    degs[5:9] = [0, 700, 33, 64]
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    items = (n_rows + len(col) + 31) // 32
    assert len(col) < 6 * n_rows and (items * dim >= 300_000) == joined and len(col) < 100_000
    halo, bits, off, packed, params, H_plain, H_ref = _packed_case(oracle, rng, n_cols, 1_000, dim, ld, seed=6)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)
    H[:, :dim] = H_ref
    once = _check_spmm(oracle, rowptr, col, val, 0, n_rows, H, dim, ldo=ld)
    assert np.array_equal(once.view(np.uint32), _gpu_spmm(rowptr, col, val, 0, n_rows, H, dim, ldo=ld).view(np.uint32))
    fused = _gpu_spmm_packed(rowptr, col, val, 0, n_rows, H_plain, dim, B.adaqp_plan_slot_of_row(n_cols, halo), packed, params, bits, off, ld)
    assert np.array_equal(once.view(np.uint32), fused.view(np.uint32))


@pytest.mark.parametrize("dim,ldh", [(128, 128), (602, 608), (602, 602), (300, 300), (7, 7), (1, 1), (66, 66),
                                     (130, 132), (250, 256), (2049, 2080), (2304, 2304), (4100, 4100), (515, 515)])
def test_spmm_packed_rows(oracle, dim, ldh):
    _say(f"spmm from packed rows dim={dim} ldh={ldh}")
    rng = np.random.default_rng(1000 + dim)
    n_rows, n_cols, n_halo = 500, 700, 330
    degs = rng.integers(0, 12, size=n_rows)
    degs[10] = 650                                                     # split over several pieces
    degs[300:310] = 0
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    halo, bits, off, packed, params, H_plain, H_ref = _packed_case(oracle, rng, n_cols, n_halo, dim, ldh, seed=77)
    slot_of_row = B.adaqp_plan_slot_of_row(n_cols, halo)
    assert np.array_equal(np.nonzero(slot_of_row >= 0)[0], np.sort(halo))
    assert np.array_equal(halo[slot_of_row[np.sort(halo)]], np.sort(halo))
    ldo = ldh if ldh % 32 == 0 else dim
    got = _gpu_spmm_packed(rowptr, col, val, 0, n_rows, H_plain, dim, slot_of_row, packed, params, bits, off, ldo)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, H_ref, dim)
    err = np.abs(got[:, :dim].astype(np.float64) - want)
    worst = float((err / (SPMM_RTOL * mag + 1e-30)).max())
    assert worst <= 1.0, f"worst error {worst:.3f} x tolerance"
    zero_to = _padded_cols(dim, ldo) if (ldo % 32 == 0 and ldh % 32 == 0) else dim
    assert np.all(got[:, dim:zero_to] == 0.0) and np.all(got[:, zero_to:] == 7.0)
    # bit-identical to de-quantising into H first (same arithmetic, same order)
    H_filled = np.full((n_cols, ldh), np.nan, dtype=np.float32)
    H_filled[:, :dim] = H_ref
    unfused = _gpu_spmm(rowptr, col, val, 0, n_rows, H_filled, dim, ldo=ldo)
    assert np.array_equal(got.view(np.uint32), unfused.view(np.uint32))
    # a sub-range, and a map with unusable slots: those entries read H
    sub = _gpu_spmm_packed(rowptr, col, val, 9, 12, H_plain, dim, slot_of_row, packed, params, bits, off, ldo)
    sub_unfused = _gpu_spmm(rowptr, col, val, 9, 12, H_filled, dim, ldo=ldo)      # same pieces, same order
    assert np.array_equal(sub.view(np.uint32), sub_unfused.view(np.uint32)) and np.all(sub[:9] == 7.0)
    broken = slot_of_row.copy()
    broken[halo[:50]] = n_halo + 5
    H_mixed = H_plain.copy()
    H_mixed[halo[:50], :dim] = H_ref[halo[:50]]
    again = _gpu_spmm_packed(rowptr, col, val, 0, n_rows, H_mixed, dim, broken, packed, params, bits, off, ldo)
    assert np.array_equal(again.view(np.uint32), got.view(np.uint32))


@pytest.mark.parametrize("dim,ldh,n_cols,rows,mean", [
    # whole lines, all of the matrix in the L2s: slices of four lines and what may be left over, of two lines
    (32, 32, 700, 1500, 80), (96, 96, 700, 1500, 80), (128, 160, 700, 1500, 80), (150, 160, 700, 1500, 80),
    (192, 192, 700, 1500, 80), (224, 224, 700, 1500, 80), (288, 288, 700, 1500, 120), (300, 320, 700, 1500, 80),
    (410, 416, 700, 1500, 120), (512, 544, 700, 1500, 50), (480, 480, 700, 1500, 400),
    # slices of one line (packed: four) and half shares, of two lines, of two lines (packed: four)
    (60, 64, 50_000, 1500, 80), (100, 128, 50_000, 1500, 80), (224, 224, 50_000, 1500, 80), (640, 640, 41_000, 3000, 180),
    (64, 64, 201_000, 1500, 80), (250, 256, 201_000, 1500, 80), (620, 640, 201_000, 4000, 420),
    # rows that share lines: narrow ones, long ones
    (5, 7, 700, 1500, 80), (33, 33, 700, 1500, 80), (64, 65, 700, 1500, 80), (66, 66, 700, 1500, 100),
    (97, 98, 700, 1500, 100), (131, 131, 700, 1500, 100), (301, 302, 700, 1500, 100), (515, 517, 700, 1500, 100)])
def test_spmm_cuts(oracle, dim, ldh, n_cols, rows, mean):
    """Entries enough for the sliced kernel in each of its cuts, plain and from packed rows: row ends at every place of a step,
    more row ends than a chunk takes, rows of many shares' length, empty rows at both ends; the same bits packed."""
    _say(f"spmm cut dim={dim} ldh={ldh} n_cols={n_cols} mean={mean}")
    rng = np.random.default_rng(dim + n_cols)
    degs = np.concatenate([np.zeros(70), np.ones(130), np.arange(40), [383, 384, 385, 8, 16, 0, 0], np.full(60, 23),
                           [20_000, 5, 3_000], rng.integers(mean // 2, mean * 3 // 2 + 1, size=rows), np.zeros(3)]).astype(int)
    n_rows = degs.shape[0]
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    assert len(col) >= (60_000 if dim == 512 else (150_000 if dim in (288, 410) else 100_000))
    halo, bits, off, packed, params, H_plain, H_ref = _packed_case(oracle, rng, n_cols, min(n_cols // 2, 3000), dim, ldh, seed=7)
    slot_of_row = B.adaqp_plan_slot_of_row(n_cols, halo)
    H_filled = np.full((n_cols, ldh), np.nan, dtype=np.float32)     # what lies between the rows must never reach a sum
    H_filled[:, :dim] = H_ref
    ldo = ldh if ldh % 32 == 0 else dim
    got = _check_spmm(oracle, rowptr, col, val, 0, n_rows, H_filled, dim, ldo=ldo)
    _check_spmm(oracle, rowptr, col, val, 65, n_rows - 1, H_filled, dim, nnz_range="exact", ldo=ldo)
    fused = _gpu_spmm_packed(rowptr, col, val, 0, n_rows, H_plain, dim, slot_of_row, packed, params, bits, off, ldo)
    assert np.array_equal(fused.view(np.uint32), got.view(np.uint32))


def test_spmm_packed_argument_checks():
    z = torch.zeros(64, dtype=torch.uint8, device=DEV)
    rowptr = torch.zeros(2, dtype=torch.int64, device=DEV)
    col = torch.zeros(1, dtype=torch.int32, device=DEV)[:0]
    val = torch.zeros(1, dtype=torch.float32, device=DEV)[:0]
    H = torch.zeros((4, 32), dtype=torch.float32, device=DEV)
    out = torch.zeros((1, 32), dtype=torch.float32, device=DEV)
    slot = torch.full((4,), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.AdaqpError):                      # a map without slots
        B.adaqp_spmm_csr_packed(rowptr, col, val, 0, 1, H, 32, out, slot, z, torch.zeros((1, 2), device=DEV),
                                z[:0], torch.zeros(1, dtype=torch.int64, device=DEV)[:0], ws)


# ------------------------------------------------------------------------------------------------------
# aggregation tiled over the L2 caches (long rows)
# ------------------------------------------------------------------------------------------------------

def _gpu_spmm_tiled(rowptr, col, val, rb, re, H, dim, ldo, chunk_cols=0):
    n_cols = H.shape[0]
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
    out = torch.full((rowptr.shape[0] - 1, ldo), 7.0, dtype=torch.float32, device=DEV)
    ws = torch.empty(max(B.adaqp_spmm_tiled_workspace_bytes(re - rb, dim), 256), dtype=torch.uint8, device=DEV)
    ws.fill_(0xFF)                                              # NaN patterns: unread unless written first
    B.adaqp_spmm_csr_tiled(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV),
                           torch.from_numpy(val).to(DEV), rb, re, torch.from_numpy(H).to(DEV), dim, out,
                           torch.from_numpy(off).to(DEV), ws, chunk_cols=chunk_cols)
    torch.cuda.synchronize()
    return out.cpu().numpy(), bounds, off


@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (64, 64), (7, 32), (60, 64), (96, 96), (100, 128),
                                    (130, 160), (256, 256), (2049, 2080)])
def test_spmm_tiled(oracle, dim, ld):
    _say(f"tiled spmm dim={dim} ld={ld}")
    rng = np.random.default_rng(2000 + dim)
    n_rows, n_cols = 300, 900
    degs = rng.integers(0, 150, size=n_rows)
    degs[10] = 880                                                     # nearly every column
    degs[11] = 0
    degs[100:110] = 0
    degs[200:230] = rng.integers(1, 4, size=30)                        # rows that miss most tiles
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)                # NaN in the row padding
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    got, bounds, off = _gpu_spmm_tiled(rowptr, col, val, 0, n_rows, H, dim, ld)
    # the plan: tiles cover the columns, hold about an eighth of the entries each, and count each row's entries
    assert bounds[0] == 0 and bounds[-1] == col.max() + 1 and np.all(np.diff(bounds) >= 0)
    per_tile = np.histogram(col, bins=bounds.astype(np.int64))[0] if False else \
        np.array([np.count_nonzero((col >= bounds[t]) & (col < bounds[t + 1])) for t in range(B.SPMM_TILES)])
    assert per_tile.sum() == len(col) and per_tile.max() <= len(col) / B.SPMM_TILES + degs.max()
    for r in (0, 10, 11, 205, 299):
        c = col[rowptr[r]: rowptr[r + 1]]
        if len(c) >= B.SPMM_TILED_SHORT_ROW:
            assert [int(np.count_nonzero(c < b)) for b in bounds] == off[r].tolist()
        else:                                                          # short rows stay whole, in one tile
            assert off[r].tolist() == [0 if t <= r % B.SPMM_TILES else len(c) for t in range(B.SPMM_TILES + 1)]
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    err = np.abs(got[:, :dim].astype(np.float64) - want)
    worst = float((err / (SPMM_RTOL * mag + 1e-30)).max())
    assert worst <= 1.0, f"worst error {worst:.3f} x tolerance"
    zero_to = _padded_cols(dim, ld)
    assert np.all(got[:, dim:zero_to] == 0.0) and np.all(got[:, zero_to:] == 7.0)
    again, _, _ = _gpu_spmm_tiled(rowptr, col, val, 0, n_rows, H, dim, ld)
    assert np.array_equal(got.view(np.uint32), again.view(np.uint32)), "runs differ"
    assert B.adaqp_spmm_tiled_chunk_cols(bounds, dim) == (64 if dim <= 96 else 128)     # ranges of ~110 columns
    narrow, _, _ = _gpu_spmm_tiled(rowptr, col, val, 0, n_rows, H, dim, ld, chunk_cols=64)
    err = np.abs(narrow[:, :dim].astype(np.float64) - want)
    assert np.all(err <= SPMM_RTOL * mag + 1e-30), "64-column chunks"
    assert np.all(narrow[:, dim:zero_to] == 0.0) and np.all(narrow[:, zero_to:] == 7.0)
    none, _, _ = _gpu_spmm_tiled(rowptr, col, val, 100, 110, H, dim, ld)           # a range of empty rows only
    assert np.all(none[100:110, :zero_to] == 0.0) and np.all(none[:100] == 7.0) and np.all(none[110:] == 7.0)
    sub, _, _ = _gpu_spmm_tiled(rowptr, col, val, 9, 120, H, dim, ld)
    assert np.all(sub[:9] == 7.0) and np.all(sub[120:] == 7.0)
    err = np.abs(sub[9:120, :dim].astype(np.float64) - want[9:120])
    assert np.all(err <= SPMM_RTOL * mag[9:120] + 1e-30)


def test_spmm_tiled_random_shapes(oracle):
    """Seeded sweep over small shapes: fewer columns than tiles, single rows, one dense row, ragged widths."""
    rng = np.random.default_rng(4242)
    dims = [1, 5, 31, 32, 33, 64, 65, 127, 128, 129, 200, 256, 300, 602]
    for case in range(24):
        n_rows = int(rng.choice([1, 2, 3, 15, 16, 17, 100, 257]))
        n_cols = int(rng.choice([1, 2, 7, 8, 9, 70, 500, 1500]))
        dim = int(rng.choice(dims))
        ld = (dim + 31) // 32 * 32
        kind = case % 4
        if kind == 0:
            degs = rng.integers(0, min(n_cols, 200) + 1, size=n_rows)
        elif kind == 1:
            degs = np.full(n_rows, n_cols)                              # dense
        elif kind == 2:
            degs = np.zeros(n_rows, dtype=np.int64)
            degs[rng.integers(0, n_rows)] = n_cols                      # one full row, the rest empty
        else:
            degs = rng.integers(0, 3, size=n_rows)                      # nearly empty
        _say(f"tiled spmm case {case}: rows {n_rows} cols {n_cols} dim {dim} kind {kind}")
        rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
        H = np.full((n_cols, ld), np.nan, dtype=np.float32)
        H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
        want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
        for chunk in (0, 64):
            if len(col) == 0:
                # no entries at all: col / val may not even exist; the call only has to zero the rows
                got = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
                off = np.zeros((n_rows, B.SPMM_TILES + 1), dtype=np.int32)
                ws = torch.empty(max(B.adaqp_spmm_tiled_workspace_bytes(n_rows, dim), 256), dtype=torch.uint8,
                                 device=DEV)
                B.adaqp_spmm_csr_tiled(torch.from_numpy(rowptr).to(DEV), torch.zeros(1, dtype=torch.int32, device=DEV)[:0],
                                       torch.zeros(1, dtype=torch.float32, device=DEV)[:0], 0, n_rows,
                                       torch.from_numpy(H).to(DEV), dim, got, torch.from_numpy(off).to(DEV), ws,
                                       chunk_cols=chunk)
                torch.cuda.synchronize()
                got = got.cpu().numpy()
            else:
                got, _, _ = _gpu_spmm_tiled(rowptr, col, val, 0, n_rows, H, dim, ld, chunk_cols=chunk)
            err = np.abs(got[:, :dim].astype(np.float64) - want)
            assert np.all(err <= SPMM_RTOL * mag + 1e-30), f"case {case} chunk {chunk}"
            assert np.all(got[:, dim:] == 0.0), f"case {case}: row padding"


def test_spmm_tiled_rejects_what_it_cannot_do():
    rowptr = np.array([0, 2], dtype=np.int64)
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_tiles(rowptr, np.array([3, 1], dtype=np.int32), 0, 1, 8)        # not ascending
    with pytest.raises(B.AdaqpError):
        B.adaqp_plan_spmm_tiles(rowptr, np.array([1, 9], dtype=np.int32), 0, 1, 8)        # out of range
    _, off = B.adaqp_plan_spmm_tiles(rowptr, np.array([1, 3], dtype=np.int32), 0, 1, 8)
    H = torch.zeros((8, 30), dtype=torch.float32, device=DEV)                              # pitch not whole lines
    out = torch.zeros((1, 30), dtype=torch.float32, device=DEV)
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.AdaqpError):
        B.adaqp_spmm_csr_tiled(torch.from_numpy(rowptr).to(DEV), torch.tensor([1, 3], dtype=torch.int32, device=DEV),
                               torch.ones(2, device=DEV), 0, 1, H, 30, out, torch.from_numpy(off).to(DEV), ws)


# ------------------------------------------------------------------------------------------------------
# dense panels of the longest rows on the matrix cores, the tiled kernel for the rest
# ------------------------------------------------------------------------------------------------------

def _gpu_spmm_tiled_and_panels(rowptr, col, val, rb, re, H, dim, ldo, min_row_len, piece_cols, chunk_cols=0):
    n_cols = H.shape[0]
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
    plan = B.adaqp_plan_spmm_panels(rowptr, col, val, rb, re, n_cols, bounds, off, min_row_len, piece_cols)
    panels = B.DevicePanels(plan, DEV)
    out = torch.full((rowptr.shape[0] - 1, ldo), 7.0, dtype=torch.float32, device=DEV)
    nbytes = max(B.adaqp_spmm_tiled_workspace_bytes(re - rb, dim),
                 B.adaqp_spmm_panels_workspace_bytes(panels.n_per_tile, dim), 256)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    ws.fill_(0xFF)                                              # NaN patterns: unread unless written first
    Hd = torch.from_numpy(H).to(DEV)
    B.adaqp_spmm_csr_tiled(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV),
                           torch.from_numpy(val).to(DEV), rb, re, Hd, dim, out, torch.from_numpy(off).to(DEV), ws,
                           chunk_cols=chunk_cols)
    ws.fill_(0xFF)
    B.adaqp_spmm_csr_panels(panels, rb, re, Hd, dim, out, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy(), plan


@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (64, 64), (7, 32), (100, 128), (130, 160), (256, 256),
                                    (1025, 1056)])
def test_spmm_panels(oracle, dim, ld):
    _say(f"panel spmm dim={dim} ld={ld}")
    rng = np.random.default_rng(3000 + dim)
    n_rows, n_cols = 300, 900
    degs = rng.integers(0, 90, size=n_rows)
    heavy = rng.choice(n_rows, size=70, replace=False)                 # two full panels and a part of a third
    degs[heavy] = rng.integers(100, 600, size=70)
    degs[heavy[0]] = n_cols                                            # every column
    degs[heavy[1]] = 100                                               # exactly the threshold
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)                # NaN in the row padding
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    zero_to = _padded_cols(dim, ld)
    first = None
    for piece_cols in (8, 64, 1024):
        got, plan = _gpu_spmm_tiled_and_panels(rowptr, col, val, 0, n_rows, H, dim, ld, 100, piece_cols)
        assert plan["n_rows_taken"] == int(np.count_nonzero(degs >= 100)) == 70 and plan["n_panels"] == 3
        err = np.abs(got[:, :dim].astype(np.float64) - want)
        worst = float((err / (SPMM_RTOL * mag + 1e-30)).max())
        assert worst <= 1.0, f"piece_cols {piece_cols}: worst error {worst:.3f} x tolerance"
        assert np.all(got[:, dim:zero_to] == 0.0) and np.all(got[:, zero_to:] == 7.0)
        if first is None:
            first = got
    again, _ = _gpu_spmm_tiled_and_panels(rowptr, col, val, 0, n_rows, H, dim, ld, 100, 8)
    assert np.array_equal(first.view(np.uint32), again.view(np.uint32)), "runs differ"
    # a sub-range: rows outside stay untouched, also those that would be long enough
    sub, plan = _gpu_spmm_tiled_and_panels(rowptr, col, val, 40, 210, H, dim, ld, 100, 64)
    assert plan["n_rows_taken"] == int(np.count_nonzero(degs[40:210] >= 100))
    assert np.all(sub[:40] == 7.0) and np.all(sub[210:] == 7.0)
    err = np.abs(sub[40:210, :dim].astype(np.float64) - want[40:210])
    assert np.all(err <= SPMM_RTOL * mag[40:210] + 1e-30)
    # the panels alone write the rows they list and nothing else
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
    plan = B.adaqp_plan_spmm_panels(rowptr, col, val, 0, n_rows, n_cols, bounds, off, 100, 64)
    panels = B.DevicePanels(plan, DEV)
    out = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
    ws = torch.empty(B.adaqp_spmm_panels_workspace_bytes(panels.n_per_tile, dim), dtype=torch.uint8, device=DEV)
    B.adaqp_spmm_csr_panels(panels, 0, n_rows, torch.from_numpy(H).to(DEV), dim, out, ws)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    listed = np.zeros(n_rows, dtype=bool)
    listed[plan["panel_rows"][plan["panel_rows"] >= 0]] = True
    assert np.all(out[~listed] == 7.0)
    err = np.abs(out[listed, :dim].astype(np.float64) - want[listed])
    assert np.all(err <= SPMM_RTOL * mag[listed] + 1e-30)
    # ... and the tiled kernel leaves exactly those rows alone, so the two may run at the same time: on two
    # streams, a workspace each, the bits are those of one after the other
    rp, cl, vl = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, val))
    Hd, offd = torch.from_numpy(H).to(DEV), torch.from_numpy(off).to(DEV)
    ws_t = torch.empty(B.adaqp_spmm_tiled_workspace_bytes(n_rows, dim), dtype=torch.uint8, device=DEV)
    only_tiled = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
    B.adaqp_spmm_csr_tiled(rp, cl, vl, 0, n_rows, Hd, dim, only_tiled, offd, ws_t)
    torch.cuda.synchronize()
    assert torch.all(only_tiled[torch.from_numpy(listed).to(DEV)] == 7.0)
    one_after_the_other = only_tiled.clone()
    B.adaqp_spmm_csr_panels(panels, 0, n_rows, Hd, dim, one_after_the_other, ws)
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)
    together = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    B.adaqp_spmm_csr_panels(panels, 0, n_rows, Hd, dim, together, ws, stream=s2)
    B.adaqp_spmm_csr_tiled(rp, cl, vl, 0, n_rows, Hd, dim, together, offd, ws_t, stream=s1)
    s1.synchronize()
    s2.synchronize()
    assert torch.equal(together.view(torch.int32), one_after_the_other.view(torch.int32))


def test_non_finite_neighbour_row_and_the_aggregation_paths(oracle):
    """Inputs must be finite.  What happens otherwise is pinned here so that it cannot change unnoticed: an Inf in
    one row of H reaches exactly the rows that have an edge to it in the merge-path and tiled kernels (Sec. 2.1
    Eq. 3 sums over a row's own neighbours); the dense panels multiply every row of H they list by all 32
    coefficients of a panel column, zeros included, so there it reaches every row of the panels that list the
    column (0 * Inf = NaN) - and no row outside them."""
    _say("non-finite row")
    rng = np.random.default_rng(77)
    n_rows, n_cols, dim, ld = 200, 640, 64, 64
    degs = rng.integers(2, 40, size=n_rows)
    heavy = rng.choice(n_rows, size=40, replace=False)
    degs[heavy] = rng.integers(150, 400, size=40)
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = rng.standard_normal((n_cols, ld), dtype=np.float32)
    bad_col = int(col[rowptr[heavy[0]]])                       # a column that a panel row references
    H[bad_col, 3] = np.inf
    has_edge = np.array([bad_col in col[rowptr[r]: rowptr[r + 1]] for r in range(n_rows)])
    assert has_edge.any() and not has_edge.all()
    merge = _gpu_spmm(rowptr, col, val, 0, n_rows, H, dim)
    tiled, _, _ = _gpu_spmm_tiled(rowptr, col, val, 0, n_rows, H, dim, ld)
    for name, got in (("merge path", merge), ("tiled", tiled)):
        bad_rows = ~np.isfinite(got[:, :dim]).all(axis=1)
        assert np.array_equal(bad_rows, has_edge), name
        assert np.isfinite(got[:, [c for c in range(dim) if c != 3]]).all(), name     # only the column of the Inf
    both, plan = _gpu_spmm_tiled_and_panels(rowptr, col, val, 0, n_rows, H, dim, ld, 150, 64)
    bad_rows = ~np.isfinite(both[:, :dim]).all(axis=1)
    assert np.all(bad_rows[has_edge])                          # never fewer rows than the definition
    panel_rows = plan["panel_rows"].reshape(-1, 32)
    listing = np.zeros(n_rows, dtype=bool)
    for rows in panel_rows:
        rows = rows[rows >= 0]
        if any(bad_col in col[rowptr[r]: rowptr[r + 1]] for r in rows):
            listing[rows] = True
    assert np.array_equal(bad_rows, has_edge | listing)


def test_spmm_panels_random_shapes(oracle):
    """Seeded sweep over small shapes: fewer columns than tiles, a single long row, dense blocks, ragged widths."""
    rng = np.random.default_rng(777)
    dims = [1, 5, 31, 32, 33, 64, 127, 128, 129, 200, 300, 602]
    for case in range(20):
        n_rows = int(rng.choice([1, 2, 31, 32, 33, 65, 150]))
        n_cols = int(rng.choice([1, 3, 7, 8, 9, 70, 500, 1500]))
        dim = int(rng.choice(dims))
        ld = (dim + 31) // 32 * 32
        kind = case % 4
        if kind == 0:
            degs = rng.integers(0, min(n_cols, 300) + 1, size=n_rows)
        elif kind == 1:
            degs = np.full(n_rows, n_cols)                              # dense
        elif kind == 2:
            degs = rng.integers(0, 3, size=n_rows)
            degs[rng.integers(0, n_rows)] = n_cols                      # one full row among nearly empty ones
        else:
            degs = np.where(rng.random(n_rows) < 0.3, n_cols // 2 + 1, 1)
        min_len = int(rng.choice([1, 2, 4, 50]))
        piece_cols = int(rng.choice([8, 16, 256]))
        _say(f"panel spmm case {case}: rows {n_rows} cols {n_cols} dim {dim} kind {kind} min {min_len} piece {piece_cols}")
        rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
        if len(col) == 0:
            continue
        H = np.full((n_cols, ld), np.nan, dtype=np.float32)
        H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
        want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
        got, plan = _gpu_spmm_tiled_and_panels(rowptr, col, val, 0, n_rows, H, dim, ld, min_len, piece_cols)
        assert (plan is None) == (not np.any(np.diff(rowptr) >= min_len))
        err = np.abs(got[:, :dim].astype(np.float64) - want)
        assert np.all(err <= SPMM_RTOL * mag + 1e-30), f"case {case}"
        assert np.all(got[:, dim:] == 0.0), f"case {case}: row padding"


def test_spmm_panels_rejects_what_it_cannot_do():
    rng = np.random.default_rng(5)
    rowptr, col, val = _random_graph(rng, 40, 64, np.full(40, 20))
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, 40, 64)
    panels = B.DevicePanels(B.adaqp_plan_spmm_panels(rowptr, col, val, 0, 40, 64, bounds, off, 10, 16), DEV)
    assert panels and panels.c.n_panels == 2
    need = B.adaqp_spmm_panels_workspace_bytes(panels.n_per_tile, 32)
    H = torch.zeros((64, 32), dtype=torch.float32, device=DEV)
    out = torch.zeros((40, 32), dtype=torch.float32, device=DEV)
    with pytest.raises(B.AdaqpError):                                      # workspace too small
        B.adaqp_spmm_csr_panels(panels, 0, 40, H, 32, out, torch.empty(need - 256, dtype=torch.uint8, device=DEV))
    Hbad = torch.zeros((64, 40), dtype=torch.float32, device=DEV)         # pitch not whole lines
    with pytest.raises(B.AdaqpError):
        B.adaqp_spmm_csr_panels(panels, 0, 40, Hbad, 32, out, torch.empty(need, dtype=torch.uint8, device=DEV))
    empty = B.DevicePanels(None)                                           # no panels: a successful no-op
    B.adaqp_spmm_csr_panels(empty, 0, 40, H, 32, out, torch.empty(256, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    assert torch.all(out == 0)


# ------------------------------------------------------------------------------------------------------
# the layer step
# ------------------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (64, 96), (7, 32), (96, 96), (256, 288), (2049, 2080)])
@pytest.mark.parametrize("n_rows,n_cols", [(300, 900), (700, 40_000), (1, 9)])          # one group of tiles; several; one row
def test_spmm_segments(oracle, dim, ld, n_rows, n_cols):
    """Rows of none to eight segments, short ones whole in one, some struck from the table, which stay as they are."""
    _say(f"segments spmm dim={dim} ld={ld} rows={n_rows} cols={n_cols}")
    rng = np.random.default_rng(5000 + dim)
    degs = np.minimum(rng.integers(0, 130, size=n_rows), n_cols)
    degs[0] = min(n_cols, 3_000)
    if n_rows > 9:
        degs[5:9], degs[n_rows // 2] = 0, 800
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)                # NaN in the row padding
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (col, val, H))
    for rb, re in ((0, n_rows), (n_rows // 3, n_rows)):
        bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        struck = np.arange(re - rb) % 7 == 3
        off[struck] = -1
        plan = B.adaqp_plan_spmm_segments(rowptr, rb, re, bounds, off)
        segments = B.DeviceSegments(plan, DEV)
        B.adaqp_fill_spmm_segments(segments, cl, vl)
        ws = torch.empty(B.adaqp_spmm_segments_workspace_bytes(segments, dim), dtype=torch.uint8, device=DEV)
        ws.fill_(0xFF)                                                 # NaN patterns: unread unless written first
        out = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
        B.adaqp_spmm_csr_segments(segments, rb, Hd, dim, out, ws)
        again = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
        B.adaqp_spmm_csr_segments(segments, rb, Hd, dim, again, ws)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), again.view(torch.int32))
        got = out.cpu().numpy()
        mine = np.zeros(n_rows, dtype=bool)
        mine[rb:re] = ~struck
        err = np.abs(got[mine][:, :dim].astype(np.float64) - want[mine])
        worst = float((err / (SPMM_RTOL * mag[mine] + 1e-30)).max())
        assert worst <= 1.0, f"worst error {worst:.3f} x tolerance"
        zero_to = _padded_cols(dim, ld)
        assert np.all(got[mine][:, dim:zero_to] == 0.0) and np.all(got[mine][:, zero_to:] == 7.0) and np.all(got[~mine] == 7.0)


@pytest.mark.parametrize("lines", [1, 2, 4])
@pytest.mark.parametrize("dim,ld", [(7, 32), (64, 96), (96, 96), (128, 128), (602, 608), (2049, 2080)])
def test_spmm_pieces(oracle, lines, dim, ld):
    """Segments in planned pieces: of none, one and many entries, cut by pieces, more ends than a piece takes, in rows of several segments,
    of one, struck ones; the sums of the same segments cut on the device."""
    _say(f"pieces spmm lines={lines} dim={dim} ld={ld}")
    rng = np.random.default_rng(6000 + dim)
    n_rows, n_cols = 420, 40_000
    degs = rng.integers(0, 130, size=n_rows)
    degs[:100], degs[100:110], degs[110], degs[111], degs[112] = 1, [0, 1, 7, 8, 9, 63, 64, 255, 256, 257], 9_000, 767, 769
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (col, val, H))
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, 0, n_rows, n_cols)
    struck = np.arange(n_rows) % 7 == 3
    off[struck] = -1
    plan = B.adaqp_plan_spmm_segments(rowptr, 0, n_rows, bounds, off)
    cut = B.DeviceSegments(plan, DEV)
    plan["pieces"] = B.adaqp_plan_spmm_pieces(plan["ptr"], plan["of_row"], dim, lines)
    assert (plan["pieces"]["dest"] < 0).any() and (plan["pieces"]["pieces"]["partial"] != -1).any()
    segments = B.DeviceSegments(plan, DEV)
    B.adaqp_fill_spmm_segments(segments, cl, vl)
    ws = torch.empty(max(B.adaqp_spmm_segments_workspace_bytes(segments, dim), 1), dtype=torch.uint8, device=DEV)
    outs = []
    for _ in range(2):
        ws.fill_(0xFF)
        outs.append(torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV))
        B.adaqp_spmm_csr_segments(segments, 0, Hd, dim, outs[-1], ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    got = outs[0].cpu().numpy()
    err = np.abs(got[~struck][:, :dim].astype(np.float64) - want[~struck])
    assert float((err / (SPMM_RTOL * mag[~struck] + 1e-30)).max()) <= 1.0
    zero_to = _padded_cols(dim, ld)
    assert np.all(got[~struck][:, dim:zero_to] == 0.0) and np.all(got[~struck][:, zero_to:] == 7.0) and np.all(got[struck] == 7.0)
    B.adaqp_fill_spmm_segments(cut, cl, vl)
    ws = torch.empty(max(B.adaqp_spmm_segments_workspace_bytes(cut, dim), 1), dtype=torch.uint8, device=DEV)
    B.adaqp_spmm_csr_segments(cut, 0, Hd, dim, outs[1].fill_(7.0), ws)
    torch.cuda.synchronize()
    shares = outs[1].cpu().numpy()                                     # either is off by no more than the bound
    assert np.all(np.abs(got[:, :dim].astype(np.float64) - shares[:, :dim])[~struck] <= 2 * SPMM_RTOL * mag[~struck] + 1e-30)
    assert np.array_equal(got[:, dim:], shares[:, dim:]) and np.array_equal(got[struck], shares[struck])


@pytest.mark.parametrize("lines", [1, 2, 4])
@pytest.mark.parametrize("n_rows,long,dim", [(1, 1, 40), (90, 700, 40), (300, 3_000, 100), (9_000, 30_000, 129), (60_000, 30_000, 129)])
def test_spmm_pieces_of_rows(oracle, lines, n_rows, long, dim):
    """Pieces over the rows of a CSR from the middle of its arrays on: rows without entries, parts of a row joined in a workgroup or added up
    afterwards, short and long pieces."""
    _say(f"pieces of rows lines={lines} rows={n_rows} dim={dim}")
    rng = np.random.default_rng(n_rows)
    n_cols, ld = 35_000, (dim + 31) // 32 * 32
    degs = rng.integers(0, 40, size=n_rows)
    degs[rng.integers(0, n_rows, size=n_rows // 4 + 1)] = 0
    degs[rng.integers(0, n_rows, size=n_rows // 40 + 1)] = rng.integers(100, long + 100, size=n_rows // 40 + 1) % 5_000
    degs[0], degs[-1] = long, 300
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, np.minimum(degs, n_cols))
    H = np.zeros((n_cols, ld), dtype=np.float32)
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    H[:, dim:] = np.nan
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    before = 37                                                        # entries of rows that are not the range's
    ptr = rowptr + before
    plan = B.adaqp_plan_spmm_pieces(ptr, None, dim, lines)
    on = {k: torch.from_numpy(v).to(DEV) for k, v in (("ptr", ptr), ("col", np.concatenate([np.full(before, -1, np.int32), col])),
                                                       ("val", np.concatenate([np.full(before, np.nan, np.float32), val])))}
    segments, pieces = B.DeviceSegments(None), B.DevicePieces(plan, DEV)
    segments.c = B.SpmmSegments(n_rows, on["col"].numel(), n_rows, on["ptr"].data_ptr(), on["ptr"].data_ptr(), on["ptr"].data_ptr(),
                                on["col"].data_ptr(), on["val"].data_ptr(), pieces.c)
    Hd, outs = torch.from_numpy(H).to(DEV), []
    ws = torch.empty(max(B.adaqp_spmm_segments_workspace_bytes(segments, dim), 256), dtype=torch.uint8, device=DEV)
    for _ in range(2):
        ws.fill_(0xFF)
        outs.append(torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV))
        B.adaqp_spmm_csr_segments(segments, 0, Hd, dim, outs[-1], ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    got = outs[0].cpu().numpy()
    assert float((np.abs(got[:, :dim].astype(np.float64) - want) / (SPMM_RTOL * mag + 1e-30)).max()) <= 1.0
    assert np.all(got[:, dim:] == 0.0)


def test_spmm_segments_of_more_rows_than_a_launch_has_waves():
    """2^26 rows and more: a wave each would be 2^32 threads."""
    _say("segments of 2^26 rows")
    n_rows, dim = (1 << 26) + 100, 32
    rng = np.random.default_rng(13)
    ptr, cols = np.array([0, 2, 3, 5, 8], np.int64), np.array([0, 3, 1, 0, 2, 1, 2, 3], np.int32)
    val, H = rng.standard_normal(8).astype(np.float32), rng.standard_normal((4, dim)).astype(np.float32)
    of_row = torch.full((n_rows, B.SPMM_SEGMENTS), -1, dtype=torch.int32, device=DEV)
    first, last = 12345, (1 << 26) + 7                                  # rows with segments, and one that is someone else's
    of_row[first, 0], of_row[last, 0], of_row[last, 5], of_row[n_rows - 1, 0] = 2, 0, 3, -2
    on = {k: torch.from_numpy(v).to(DEV) for k, v in (("ptr", ptr), ("col", cols), ("val", val))}
    segments = B.DeviceSegments(None)
    segments.c = B.SpmmSegments(4, 8, n_rows, on["ptr"].data_ptr(), on["ptr"].data_ptr(), of_row.data_ptr(), on["col"].data_ptr(),
                                on["val"].data_ptr())
    out = torch.full((n_rows, dim), 7.0, device=DEV)
    B.adaqp_spmm_csr_segments(segments, 0, torch.from_numpy(H).to(DEV), dim, out,
                              torch.empty(B.adaqp_spmm_segments_workspace_bytes(segments, dim), dtype=torch.uint8, device=DEV))
    terms = val.astype(np.float64)[:, None] * H[cols]
    for row, parts in ((first, [2]), (last, [0, 3])):
        entries = np.concatenate([terms[ptr[s]:ptr[s + 1]] for s in parts])
        assert np.all(np.abs(out[row].cpu().numpy() - entries.sum(0)) <= SPMM_RTOL * np.abs(entries).sum(0))
        out[row] = 0.0
    assert bool((out[-1] == 7.0).all())
    out[-1] = 0.0
    assert not bool(out.any())


@pytest.mark.parametrize("dim,ld", [(128, 128), (602, 608), (64, 64), (7, 32), (96, 96), (130, 160), (256, 288), (1025, 1056)])
@pytest.mark.parametrize("n_rows,n_heavy,n_cols", [(300, 140, 900), (40, 3, 33), (150, 128, 5_000)])
def test_spmm_blocks(oracle, dim, ld, n_rows, n_heavy, n_cols):
    """Blocks of 128 rows, full and partly filled, one to 4 column tiles in the last chunk, steps that the columns do not fill,
    with the tiled kernel for the other rows; then the blocks alone, which write the rows they list and nothing else."""
    _say(f"blocks spmm dim={dim} ld={ld} rows={n_rows} heavy={n_heavy} cols={n_cols}")
    rng = np.random.default_rng(4000 + dim)
    degs = rng.integers(0, 20, size=n_rows)
    heavy = rng.choice(n_rows, size=n_heavy, replace=False)
    degs[heavy] = rng.integers(25, n_cols, size=n_heavy)
    degs[heavy[0]], degs[heavy[1]] = n_cols, 25                        # every column; exactly the threshold
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, degs)
    H = np.full((n_cols, ld), np.nan, dtype=np.float32)                # NaN in the row padding
    H[:, :dim] = rng.standard_normal((n_cols, dim), dtype=np.float32)
    want, mag = oracle.spmm_csr(rowptr, col, val, 0, n_rows, np.ascontiguousarray(H[:, :dim]), dim)
    rp, cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, val, H))
    for rb, re in ((0, n_rows), (n_rows // 3, n_rows - 1)):
        _, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
        blocks = B.DeviceBlocks(B.adaqp_plan_spmm_blocks(rowptr, col, rb, re, n_cols, dim, 25, off), DEV)
        taken = np.nonzero(degs[rb:re] >= 25)[0] + rb
        assert sorted(r for r in blocks.tensors["rows"].tolist() if r >= 0) == taken.tolist()
        B.adaqp_fill_spmm_blocks(blocks, rb, re, rp, cl, vl)
        ws = torch.empty(B.adaqp_spmm_blocks_workspace_bytes(blocks, dim), dtype=torch.uint8, device=DEV)
        out = torch.full((n_rows, ld), 7.0, dtype=torch.float32, device=DEV)
        B.adaqp_spmm_csr_blocks(blocks, rb, re, Hd, dim, out, ws)
        torch.cuda.synchronize()
        rest = np.setdiff1d(np.arange(n_rows), taken)
        assert np.all(out.cpu().numpy()[rest] == 7.0)
        first = out.clone()
        ws_t = torch.empty(B.adaqp_spmm_tiled_workspace_bytes(re - rb, dim), dtype=torch.uint8, device=DEV)
        B.adaqp_spmm_csr_tiled(rp, cl, vl, rb, re, Hd, dim, out, torch.from_numpy(off).to(DEV), ws_t)
        B.adaqp_spmm_csr_blocks(blocks, rb, re, Hd, dim, out, ws)      # the same bits again
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got[taken].view(np.uint32), first.cpu().numpy()[taken].view(np.uint32))
        err = np.abs(got[rb:re, :dim].astype(np.float64) - want[rb:re])
        worst = float((err / (SPMM_RTOL * mag[rb:re] + 1e-30)).max())
        assert worst <= 1.0, f"worst error {worst:.3f} x tolerance"
        assert np.all(got[rb:re, dim:_padded_cols(dim, ld)] == 0.0) and np.all(got[:rb] == 7.0) and np.all(got[re:] == 7.0)


def test_spmm_blocks_precision():
    """fp32 operands as three bf16: against 64 bits no worse than a running fp32 sum of as many terms as one set of sums takes
    (a piece's columns), also where the products differ by many orders of magnitude."""
    _say("blocks precision")
    rng = np.random.default_rng(8)
    n_rows, n_cols, dim = 130, 4_000, 64
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, np.full(n_rows, 3_000))
    for scale in (np.ones(n_cols), 10.0 ** rng.uniform(-6, 6, n_cols)):
        for H in (np.abs(rng.standard_normal((n_cols, dim))), rng.standard_normal((n_cols, dim))):
            H = (H * scale[:, None]).astype(np.float32)
            plan = B.adaqp_plan_spmm_blocks(rowptr, col, 0, n_rows, n_cols, dim, 1)
            blocks = B.DeviceBlocks(plan, DEV)
            rp, cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, np.abs(val), H))
            B.adaqp_fill_spmm_blocks(blocks, 0, n_rows, rp, cl, vl)
            ws = torch.empty(B.adaqp_spmm_blocks_workspace_bytes(blocks, dim), dtype=torch.uint8, device=DEV)
            out = torch.zeros((n_rows, dim), device=DEV)
            B.adaqp_spmm_csr_blocks(blocks, 0, n_rows, Hd, dim, out, ws)
            A = torch.zeros((n_rows, n_cols), dtype=torch.float64, device=DEV)
            A[torch.repeat_interleave(torch.arange(n_rows, device=DEV), rp.diff()), cl.long()] = vl.double()
            want, mag = A @ Hd.double(), A @ Hd.double().abs()
            # chains: the instructions of a piece (two per step) and the pieces, of 16 columns each at most; the parts left out
            # are less than 2^-24 of a product
            steps = plan["n_steps"] // (plan["n_blocks"] * plan["n_pieces"]) + 1
            bound = (2 * steps + plan["n_pieces"] + 8 + 1) * 2.0 ** -24
            error = float(((out.double() - want).abs() / mag).max())
            assert error <= bound, (error, bound)
            rel = float((out.double() - want).norm() / want.norm())
            assert rel <= 1.5e-7, rel                                   # a rounding per term would be sqrt(3000) of them


def test_spmm_blocks_products():
    """Single products of the operands whose parts that are left out are largest (hi rounded to nearest; hi cut off), of values that
    round to infinity in bf16, and of any others: less than 2^-24 of a product left out, the sum of the others rounded once to fp32,
    and before that where the five smaller ones are added up (2^-7 of the product, five cuts of up to 2^-23)."""
    _say("blocks products")
    rng = np.random.default_rng(12)
    x = np.concatenate([np.array([0x3F807FC0, 0x3F80FF80, 0x3F80817F, 0x3F800000, 0x3F7FFFFF], np.uint32).view(np.float32),
                        rng.standard_normal(155).astype(np.float32)])
    y = np.concatenate([x[:32], np.ldexp(x[:4], 126), [3.4e38, -3.39e38], rng.standard_normal(10)]).astype(np.float32)
    x[-20:] *= 2.0 ** -60
    y = y[None, :]
    n, dim = x.size, y.size
    H = np.repeat(y, n, axis=0)
    H[:, 32:38][np.abs(x) > 2.0 ** -50] = 1.0                          # the largest values meet small ones only
    rowptr, col = np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32)
    blocks = B.DeviceBlocks(B.adaqp_plan_spmm_blocks(rowptr, col, 0, n, n, dim, 1), DEV)
    rp, cl, vl = (torch.from_numpy(a).to(DEV) for a in (rowptr, col, x))
    Hd = torch.zeros((n, 64), device=DEV)
    Hd[:, :dim] = torch.from_numpy(H).to(DEV)
    B.adaqp_fill_spmm_blocks(blocks, 0, n, rp, cl, vl)
    out = torch.zeros((n, 64), device=DEV)
    B.adaqp_spmm_csr_blocks(blocks, 0, n, Hd, dim, out,
                            torch.empty(B.adaqp_spmm_blocks_workspace_bytes(blocks, dim), dtype=torch.uint8, device=DEV))
    want = x.astype(np.float64)[:, None] * H
    error = np.abs(out[:, :dim].cpu().numpy() - want) / np.abs(want)
    assert error.max() <= (2 + 10 * 2.0 ** -7) * 2.0 ** -24, error.max() * 2 ** 24


@pytest.mark.parametrize("zeros", [0.0, 0.3])                        # share of entries with a coefficient of 0, of either sign
def test_spmm_blocks_non_finite(zeros):
    """An infinity or NaN in H reaches the rows that list its column, and no others; next to values near the ends of fp32."""
    _say("blocks non-finite")
    rng = np.random.default_rng(9)
    n_rows, n_cols, dim = 200, 700, 330                                # two strips of 256 columns, the second partly filled
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, rng.integers(150, 600, size=n_rows))
    dropped = np.random.default_rng(90).random(val.size) < zeros
    val[dropped] = np.copysign(0.0, val[dropped])
    H = rng.standard_normal((n_cols, 352)).astype(np.float32)
    for v, c, k in ((np.inf, 3, 0), (-np.inf, 90, 17), (np.nan, 400, 256), (np.inf, 401, 329), (-np.inf, 402, 329), (5e37, 500, 40)):
        H[c, k] = v                                                    # (5e37: coefficients are up to 5, products within fp32)
    H[:, dim:] = np.nan
    plan = B.adaqp_plan_spmm_blocks(rowptr, col, 0, n_rows, n_cols, dim, 1)
    blocks = B.DeviceBlocks(plan, DEV)
    rp, cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, val, H))
    B.adaqp_fill_spmm_blocks(blocks, 0, n_rows, rp, cl, vl)
    out = torch.full((n_rows, 352), 7.0, device=DEV)
    B.adaqp_spmm_csr_blocks(blocks, 0, n_rows, Hd, dim, out,
                            torch.empty(B.adaqp_spmm_blocks_workspace_bytes(blocks, dim), dtype=torch.uint8, device=DEV))
    got = out.cpu().numpy().astype(np.float64)
    want, mag = np.zeros((n_rows, dim)), np.zeros((n_rows, dim))
    with np.errstate(invalid="ignore"):
        for r in range(n_rows):
            c, a = col[rowptr[r]:rowptr[r + 1]], val[rowptr[r]:rowptr[r + 1]].astype(np.float64)[:, None]
            x = H[c, :dim].astype(np.float64)
            want[r], mag[r] = (a * x).sum(0), np.abs(a * x).sum(0)
    fine = np.isfinite(want)
    assert 0 < fine.sum() < fine.size and np.array_equal(np.isnan(got[:, :dim]), np.isnan(want))
    assert np.array_equal(got[:, :dim][np.isinf(want)], want[np.isinf(want)])
    assert np.all(np.abs(got[:, :dim][fine] - want[fine]) <= SPMM_RTOL * mag[fine])
    assert np.all(got[:, dim:] == 0.0)


@pytest.mark.parametrize("exponent", [-60, -100, -118])
def test_spmm_blocks_small_values(exponent):
    """Values whose lower parts are denormal in bf16 (2^-110 and below), and products that are denormal themselves: next to the
    relative error, no more than a rounding of the smallest fp32 number per product."""
    _say(f"blocks small values 2^{exponent}")
    rng = np.random.default_rng(10)
    n_rows, n_cols, dim = 140, 500, 64
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, rng.integers(100, 500, size=n_rows))
    H = np.ldexp(rng.standard_normal((n_cols, dim)), exponent).astype(np.float32)
    want, mag = np.zeros((n_rows, dim)), np.zeros((n_rows, dim))
    for r in range(n_rows):
        c, a = col[rowptr[r]:rowptr[r + 1]], val[rowptr[r]:rowptr[r + 1]].astype(np.float64)[:, None]
        want[r], mag[r] = (a * H[c]).sum(0), np.abs(a * H[c]).sum(0)
    blocks = B.DeviceBlocks(B.adaqp_plan_spmm_blocks(rowptr, col, 0, n_rows, n_cols, dim, 1), DEV)
    rp, cl, vl, Hd = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, val, H))
    B.adaqp_fill_spmm_blocks(blocks, 0, n_rows, rp, cl, vl)
    out = torch.zeros((n_rows, dim), device=DEV)
    B.adaqp_spmm_csr_blocks(blocks, 0, n_rows, Hd, dim, out,
                            torch.empty(B.adaqp_spmm_blocks_workspace_bytes(blocks, dim), dtype=torch.uint8, device=DEV))
    error = np.abs(out.cpu().numpy().astype(np.float64) - want)
    worst = float((error / (SPMM_RTOL * mag + n_cols * 2.0 ** -149)).max())
    assert worst <= 1.0, worst


def _oracle_layer(oracle, p, seed):
    """Composes the oracle's pieces in the order of Sec. 3.1: quantise, exchange (identity), de-quantise,
    aggregate.  Returns (packed, params, feat_after, out64, mag64)."""
    cfg = p.cfg
    perm, off, pbp = oracle.plan_layout(cfg.dim, p.bits, p.peer_of_slot, cfg.n_peers)
    s_idx = np.ascontiguousarray(p.send_idx[perm])
    s_bits = np.ascontiguousarray(p.bits[perm])
    if not cfg.backward:
        packed, params, _ = oracle.quantize_pack(p.feat, cfg.dim, s_idx, s_bits, off, seed, int(pbp[-1]))
        feat = p.feat.copy()
        oracle.unpack_dequant(packed, params, s_bits, off, np.ascontiguousarray(p.halo_idx[perm]), cfg.dim, feat)
        out64, mag = oracle.spmm_csr(p.rowptr, p.col, p.val, 0, p.n_rows, feat, cfg.dim)
        return packed, params, feat, out64, mag
    out = np.zeros((p.n_rows, cfg.dim), dtype=np.float32)
    out64, mag = oracle.spmm_csr(p.rowptr, p.col, p.val, 0, p.n_rows, p.feat, cfg.dim, out=out)
    return None, None, None, out64, mag


def test_layer_step_follows_new_coefficients():
    """Blocks and segments keep the coefficients a second time: a caller who writes others into val gets the step of those."""
    _say("layer step, new coefficients")
    p = make_partition(replace(CONFIGS["c0"], mean_degree=1500.0))
    L = LayerStep(p, DEV, seed=5, tiled=True)
    assert L.blocks_overlap and L.segments_overlap
    L.run()
    L.synchronize()
    before = L.out.clone()
    L.val.mul_(2.0)                                                    # every product and sum is exactly twice as large
    torch.cuda.synchronize()
    for _ in range(2):
        L.run()
        L.synchronize()
        assert torch.equal(L.out, before * 2.0)
    L.val = L.val * 0.5                                                # another tensor in its place
    torch.cuda.synchronize()
    L.run()
    L.synchronize()
    assert torch.equal(L.out, before)
    L.val.data.mul_(2.0)                                               # not counted
    torch.cuda.synchronize()
    L.refresh_coefficients()
    L.run()
    L.synchronize()
    assert torch.equal(L.out, before * 2.0)
    L.val.mul_(0.5)
    torch.cuda.synchronize()
    B.adaqp_layer_step(L.desc(B.ISOLATED))                             # a descriptor
    L.synchronize()
    assert torch.equal(L.out, before)
    with torch.inference_mode():                                       # such a tensor does not count its changes
        L = LayerStep(p, DEV, seed=5, tiled=True)
        for factor in (1.0, 2.0):
            L.val.mul_(factor)
            torch.cuda.synchronize()
            L.run()
            L.synchronize()
            assert torch.equal(L.out, before * factor)


def test_step_made_in_inference_mode_copies_coefficients_when_they_change():
    """Not before every step."""
    _say("inference mode, copies")
    p = make_partition(replace(CONFIGS["c0"], mean_degree=1500.0))
    with torch.inference_mode():
        L = LayerStep(p, DEV, seed=5, tiled=True)
        assert L.blocks_overlap and L.segments_overlap
        copies, refresh = [], L.refresh_coefficients
        L.refresh_coefficients = lambda: (copies.append(1), refresh())
        for writes, want in ((0, 0), (1, 1), (0, 1), (2, 2)):
            for _ in range(writes):
                L.val.mul_(2.0)
            torch.cuda.synchronize()
            L.run()
            L.desc(B.ISOLATED)
            L.synchronize()
            assert len(copies) == want


@pytest.mark.parametrize("schedule", [B.CHAIN, B.ISOLATED])
def test_captured_step_and_new_coefficients(schedule):
    """Copies made inside a capture are made by its replays: an eager step does not count on them."""
    _say(f"captured step, new coefficients, schedule {schedule}")
    p = make_partition(replace(CONFIGS["c0"], mean_degree=1500.0))
    L = LayerStep(p, DEV, seed=5, tiled=True)
    assert L.blocks_overlap and L.segments_overlap
    L.run(schedule)
    L.synchronize()
    before = L.out.clone()
    L.val.mul_(2.0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=L.stream_msg):
        L.run(schedule)
    L.run(schedule)                                                    # before any replay
    L.synchronize()
    assert torch.equal(L.out, before * 2.0)
    for factor in (4.0, 2.0, 1.0):
        L.val.copy_(torch.from_numpy(p.val).to(DEV) * factor)
        L.out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.out, before * factor)


@pytest.mark.parametrize("schedule", [B.CHAIN, B.ISOLATED])
@pytest.mark.parametrize("fused", [False, True])
def test_replays_follow_coefficients_written_after_the_capture(schedule, fused):
    """Also where val had not been written to before it; both ranges of a step whose dependent rows read val itself."""
    _say(f"replays, new coefficients, schedule {schedule}, fused {fused}")
    p = make_partition(replace(CONFIGS["c0"], mean_degree=1500.0))
    L = LayerStep(p, DEV, seed=5, tiled=True, fused_receive=fused)
    assert L.blocks_overlap and L.segments_overlap and (fused or L.segments_dependent)
    L.run(schedule)
    L.synchronize()
    before = L.out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=L.stream_msg):
        L.run(schedule)
    for factor in (2.0, 1.0, 0.0, 4.0):
        L.val.copy_(torch.from_numpy(p.val).to(DEV) * factor)
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.out, before * factor)
    captured, L.val = L.val, L.val * 0.5                               # another tensor: eager steps follow it, replays the first
    for _ in range(2):
        L.run(schedule)
        L.synchronize()
        assert torch.equal(L.out, before * 2.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.out, before * 4.0)
    L.val = captured
    L.run(schedule)
    L.synchronize()
    assert torch.equal(L.out, before * 4.0)


def test_updates_of_the_copies_write_what_has_changed():
    """Blocks and segments brought up to date are those of a fill, wherever an entry changes: first and last of the range, zeros of
    either sign, NaN."""
    _say("updates of the copies")
    rng = np.random.default_rng(14)
    n_rows, n_cols, dim = 300, 3_000, 64
    rowptr, col, val = _random_graph(rng, n_rows, n_cols, np.where(np.arange(n_rows) < 140, 1_500, rng.integers(0, 90, size=n_rows)))
    rb, re = 3, n_rows - 2
    bounds, off = B.adaqp_plan_spmm_tiles(rowptr, col, rb, re, n_cols)
    plan = B.adaqp_plan_spmm_blocks(rowptr, col, rb, re, n_cols, dim, 1_000, off)
    entries = B.adaqp_plan_spmm_segments(rowptr, rb, re, bounds, off)
    rp, cl, vl = (torch.from_numpy(x).to(DEV) for x in (rowptr, col, val))

    def filled():
        blocks, segments = B.DeviceBlocks(plan, DEV), B.DeviceSegments(entries, DEV)
        B.adaqp_fill_spmm_blocks(blocks, rb, re, rp, cl, vl)
        B.adaqp_fill_spmm_segments(segments, cl, vl)
        return blocks, segments

    blocks, segments = filled()
    copied = vl[rowptr[rb]:rowptr[re]].clone()
    some = torch.from_numpy(rng.choice(val.size, 500, replace=False)).to(DEV)
    ends = torch.tensor([rowptr[rb], rowptr[rb + 1] - 1, rowptr[re] - 1, rowptr[140], 0, val.size - 1], device=DEV)
    for at, to in ((ends, 3.0), (some, 0.0), (some[:250], -0.0), (some[100:], 2.5), (some[::7], float("nan")), (some, -1.0)):
        vl[at] = to
        B.adaqp_update_spmm_blocks(blocks, rb, re, rp, cl, vl, copied)
        B.adaqp_update_spmm_segments(segments, vl)
        want_blocks, want_segments = filled()
        for got, want, key in ((blocks, want_blocks, "table"), (segments, want_segments, "val")):
            assert torch.equal(got.tensors[key].view(torch.int32), want.tensors[key].view(torch.int32))


@pytest.mark.parametrize("name", ["c0", "c0_backward"])
def test_layer_step_matches_oracle_in_every_schedule(oracle, name):
    _say(f"layer step {name}")
    if name == "c0":
        p = make_partition(CONFIGS["c0"])
    else:
        p = make_partition(replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))
    cfg = p.cfg
    seed = 1234
    packed_w, params_w, feat_w, out64, mag = _oracle_layer(oracle, p, seed)
    results = []
    for schedule in (B.SERIAL, B.ISOLATED, B.FREE):
        L = LayerStep(p, DEV, seed=seed, backward_receive=False)
        if not cfg.backward:
            # poison what the step must produce, so that a missing dependency shows as NaN
            L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        out = L.out.cpu().numpy()
        err = np.abs(out.astype(np.float64) - out64)
        assert np.all(err <= SPMM_RTOL * mag + 1e-30), f"schedule {schedule}: aggregation off"
        packed = L.recv_packed.cpu().numpy()[: L.plan.packed_bytes]
        params = L.recv_params.cpu().numpy()[: L.plan.n]
        if not cfg.backward:
            want_beta = oracle.trace_beta(p.feat, cfg.dim, L.plan.send_idx_host, L.alpha_sq_host)
            assert np.array_equal(L.beta.cpu().numpy().view(np.uint32), want_beta.view(np.uint32))
            assert np.array_equal(packed, packed_w)
            assert np.array_equal(params.view(np.uint32), params_w.view(np.uint32))
            assert np.array_equal(L.feat.cpu().numpy().view(np.uint32), feat_w.view(np.uint32))
        results.append((out, packed, params))
    for out, packed, params in results[1:]:
        assert np.array_equal(out.view(np.uint32), results[0][0].view(np.uint32)), "schedules disagree"
        assert np.array_equal(packed, results[0][1]) and np.array_equal(params.view(np.uint32),
                                                                        results[0][2].view(np.uint32))
    if cfg.backward:
        # the oracle quantises the GPU's own fp32 aggregate: the codes depend on every bit of the input, and
        # the aggregate is only specified to a tolerance
        L = LayerStep(p, DEV, seed=seed, backward_receive=False)
        L.run(B.SERIAL)
        L.synchronize()
        g = L.out.cpu().numpy()
        want_packed, want_params, _ = oracle.quantize_pack(g, cfg.dim, L.plan.send_idx_host, L.plan.bits_host,
                                                           L.plan.row_offset_host, seed, L.plan.packed_bytes)
        assert np.array_equal(L.recv_packed.cpu().numpy()[: L.plan.packed_bytes], want_packed)
        assert np.array_equal(L.recv_params.cpu().numpy()[: L.plan.n].view(np.uint32), want_params.view(np.uint32))
        # with the receive side switched on, the received gradients are added to the local rows in slot order:
        # the oracle adds the same received bytes to the aggregate computed above
        want_out = np.ascontiguousarray(g.copy())
        oracle.unpack_dequant_add(want_packed, want_params, L.plan.bits_host, L.plan.row_offset_host,
                                  L.plan.halo_idx_host, cfg.dim, want_out)
        assert not np.array_equal(want_out, g)
        for schedule in (B.SERIAL, B.ISOLATED, B.FREE):
            L2 = LayerStep(p, DEV, seed=seed)
            L2.out.fill_(float("nan"))
            L2.run(schedule)
            L2.synchronize()
            assert np.array_equal(L2.out.cpu().numpy().view(np.uint32), want_out.view(np.uint32)), \
                f"schedule {schedule}: backward receive differs"


def test_layer_step_fused_receive(oracle):
    """Forward step whose dependent aggregation reads the receive buffer: same output bits as the step that
    de-quantises into the feature matrix first, and the halo rows of the feature matrix stay untouched."""
    p = make_partition(CONFIGS["c0"])
    cfg = p.cfg
    seed = 1234
    _, _, _, out64, mag = _oracle_layer(oracle, p, seed)
    plain = LayerStep(p, DEV, seed=seed)
    plain.run(B.SERIAL)
    plain.synchronize()
    want = plain.out.cpu().numpy()
    for schedule in (B.SERIAL, B.ISOLATED, B.FREE):
        L = LayerStep(p, DEV, seed=seed, fused_receive=True)
        L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        out = L.out.cpu().numpy()
        assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
        assert np.array_equal(out.view(np.uint32), want.view(np.uint32)), f"schedule {schedule}"
        assert bool(torch.isnan(L.feat[cfg.n_local: cfg.n_local + cfg.n_send]).all())
        assert np.array_equal(L.recv_packed.cpu().numpy(), plain.recv_packed.cpu().numpy())


@pytest.mark.parametrize("how", ["run", "descriptor", "replay"])
@pytest.mark.parametrize("schedule", [B.CHAIN, B.ISOLATED])
def test_fused_receive_follows_what_is_written_to_the_plan(schedule, how):
    """Widths, offsets and slots written in place after the step was made: the bits of the step that de-quantises first with the same
    arrays, in a new step, with a descriptor kept from before and in replays."""
    _say(f"fused receive, arrays written in place, schedule {schedule}, {how}")
    p = make_partition(CONFIGS["c0"])
    rng = np.random.default_rng(8)
    steps = [LayerStep(p, DEV, seed=7, fused_receive=fused) for fused in (True, False)]
    assert steps[0].pieces_dependent and steps[0].pieces_both
    go = []
    for L in steps:
        if how == "replay":
            L.run(schedule)
            L.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=L.stream_msg):
                L.run(schedule)
            go.append((graph, graph.replay))
        else:
            kept = L.desc(schedule)
            go.append((kept, (lambda d=kept: B.adaqp_layer_step(d)) if how == "descriptor" else (lambda L=L: L.run(schedule))))
    halo, first = p.halo_idx[steps[0].plan.perm], None
    for _ in range(3):
        bits = rng.permutation(p.bits)
        stride = np.array([0, 0, 2, 0, 4, 0, 0, 0, 8])[bits] * p.cfg.dim // 8
        order = rng.permutation(halo)
        for L in steps:
            L.plan.bits.copy_(torch.from_numpy(bits))
            L.plan.row_offset.copy_(torch.from_numpy(np.cumsum(stride) - stride))
            L.plan.halo_idx.copy_(torch.from_numpy(order))
            if L.fused_receive:
                L.slot_of_row.copy_(torch.from_numpy(B.adaqp_plan_slot_of_row(p.feat.shape[0], order)))
            L.out.fill_(float("nan"))
            L.recv_packed.zero_()
        torch.cuda.synchronize()
        for _, step in go:
            step()
        torch.cuda.synchronize()
        assert torch.equal(steps[0].out.view(torch.int32), steps[1].out.view(torch.int32))
        first = steps[0].out.clone() if first is None else first
        want = B.adaqp_plan_packed_rows(p.feat.shape[0], order, bits, np.cumsum(stride) - stride, p.cfg.dim, steps[0].plan.packed_bytes)
        assert np.array_equal(steps[0].packed_row.cpu().numpy().view(np.uint32), want)
    assert not torch.equal(first, steps[0].out)


@pytest.mark.parametrize("rows,mean,dim,shape", [(2_000, 10, 20, (8, 256)), (2_000, 10, 40, (8, 256)), (2_000, 10, 150, (8, 256)),
                                                 (24_000, 12, 66, (4, 256)), (24_000, 8, 200, (4, 768)), (24_000, 30, 20, (4, 256)),
                                                 (24_000, 90, 33, (4, 768)), (24_000, 40, 130, (4, 768)), (24_000, 40, 224, (4, 768))])
@pytest.mark.parametrize("lines", [1, 2, 4])
def test_layer_step_in_planned_pieces(oracle, monkeypatch, rows, mean, dim, shape, lines):
    """Rows in pieces of every shape, with slices of one to four lines: against the oracle, and the same bits whether received rows are read
    from the receive buffer or from feat.  A long row whose parts are added up, columns that there are not, and an infinity and a NaN in
    rows of feat: they reach the rows that list them, and neither their neighbours in the same step nor anybody else."""
    _say(f"layer step in pieces, rows={rows} mean={mean} dim={dim} lines={lines}")
    monkeypatch.setattr(B, "adaqp_spmm_pieces_rule", lambda *args, **options: (lines, -np.inf))
    p = make_partition(replace(CONFIGS["c0"], n_local=rows, n_halo=rows // 4, n_send=rows // 5, mean_degree=float(mean), dim=dim))
    rng = np.random.default_rng(dim)
    col, n_cols = p.col.copy(), p.feat.shape[0]
    first = p.dependent_rows[0]
    lengths = np.diff(p.rowptr)
    lengths[-1] += lengths[first: first + rows // 40].sum()            # the last row takes the entries of others
    lengths[first: first + rows // 40] = 0
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    out_of_range = rng.choice(col.size, col.size // 50, replace=False)
    sent = np.isin(np.arange(n_cols), np.concatenate([p.send_idx, p.halo_idx]))
    bad = rng.choice(np.flatnonzero(~sent & (np.bincount(col, minlength=n_cols) > 0)), 6, replace=False)
    feat = p.feat.copy()
    feat[bad] = 0.0
    clean = replace(p, rowptr=rowptr, val=np.where(np.isin(np.arange(col.size), out_of_range), 0.0, p.val).astype(np.float32), feat=feat)
    _, _, _, out64, mag = _oracle_layer(oracle, clean, 5)
    col[out_of_range] = np.where(rng.random(out_of_range.size) < 0.5, -1, n_cols + 3)
    feat = p.feat.copy()
    feat[bad[:3]], feat[bad[3:]] = np.inf, np.nan
    touched = np.zeros(rows, bool)
    touched[np.repeat(np.arange(rows), np.diff(rowptr))[np.isin(col, bad)]] = True
    assert touched.any() and not touched.all()
    p, want = replace(p, rowptr=rowptr, col=col, feat=feat), None
    for fused in (False, True):
        L = LayerStep(p, DEV, seed=5, tiled=False, fused_receive=fused)
        assert L.pieces_both.c.lines_per_slice == lines and (lines != 1 or (L.pieces_both.c.waves, L.pieces_both.c.entries) == shape)
        for schedule in (B.CHAIN, B.ISOLATED):
            L.out.fill_(7.0)
            torch.cuda.synchronize()
            L.run(schedule)
            L.synchronize()
            got = L.out.cpu().numpy()
            assert np.all(np.abs(got[~touched].astype(np.float64) - out64[~touched]) <= SPMM_RTOL * mag[~touched] + 1e-30)
            assert not np.isfinite(got[touched]).any()
            want = want or {}
            kept = want.setdefault(schedule, got)
            assert np.array_equal(np.isnan(got), np.isnan(kept)) and np.array_equal(got[~touched].view(np.uint32), kept[~touched].view(np.uint32))


@pytest.mark.parametrize("dim", [641, 768])
def test_layer_step_in_planned_pieces_of_many_waves(monkeypatch, dim):
    """Enough waves for the launch of packed rows that keeps a third of them away: the bits of the step that reads what was received from feat."""
    _say(f"layer step in many pieces, dim={dim}")
    monkeypatch.setattr(B, "adaqp_spmm_pieces_rule", lambda *args, **options: (1, -np.inf))
    p, want = make_partition(replace(CONFIGS["c0"], n_local=15_000, n_halo=3_000, n_send=3_000, mean_degree=130.0, dim=dim)), None
    for fused in (False, True):
        L = LayerStep(p, DEV, seed=5, tiled=False, fused_receive=fused)
        c = L.pieces_both.c
        assert c.entries == 768 and c.n_pieces * ((dim + 127) // 128) >= 9_000 and c.lines_per_slice == 1
        L.run(B.CHAIN)
        L.synchronize()
        want = L.out.clone() if want is None else want
        assert torch.equal(L.out.view(torch.int32), want.view(torch.int32))


def test_layer_step_in_planned_pieces_of_many_waves_and_entries(monkeypatch):
    """Enough waves and entries for the launch of packed rows that keeps a third of the waves away, in slices of four lines: the bits of the step
    that reads what was received from feat."""
    _say("layer step in many pieces of many entries")
    monkeypatch.setattr(B, "adaqp_spmm_pieces_rule", lambda *args, **options: (1, -np.inf))
    p, want = make_partition(replace(CONFIGS["c0"], n_local=20_000, n_halo=3_000, n_send=3_000, mean_degree=200.0, dim=650)), None
    assert p.nnz >= 2_200_000
    for fused in (False, True):
        L = LayerStep(p, DEV, seed=5, tiled=False, fused_receive=fused)
        c = L.pieces_both.c
        assert c.entries == 768 and c.n_pieces * 6 >= 9_000 and c.lines_per_slice == 1
        L.run(B.CHAIN)
        L.synchronize()
        want = L.out.clone() if want is None else want
        assert torch.equal(L.out.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("rows,mean,dim,shape", [(2_000, 10, 128, (8, 256)), (2_000, 10, 40, (8, 256)), (24_000, 18, 66, (4, 256)),
                                                 (24_000, 60, 150, (4, 768)), (24_000, 100, 40, (4, 768))])
@pytest.mark.parametrize("kind", ["forward", "fused", "backward"])
def test_layer_step_follows_rowptr(oracle, kind, rows, mean, dim, shape):
    """Rows that were planned in pieces and whose rowptr is written to afterwards, where nobody counts that: by a descriptor kept from before,
    a replay, and a step after a write through .data.  Rows of other lengths, moved by some entries, all entries in one row, none."""
    _say(f"layer step, rowptr written in place, {kind} rows={rows} dim={dim}")
    p = make_partition(replace(CONFIGS["c0"], n_local=rows, n_halo=rows // 4, n_send=rows // 5, mean_degree=float(mean), dim=dim,
                               feat="grad" if kind == "backward" else "normal", backward=kind == "backward"))
    L = LayerStep(p, DEV, seed=3, tiled=False, fused_receive=kind == "fused", backward_receive=False)
    assert (L.pieces_both.c.waves, L.pieces_both.c.entries) == shape
    # any row may list received rows now: ranges that are aggregated before these are in place are not for a forward step
    schedules = {"forward": (B.CHAIN, B.SERIAL), "fused": (B.CHAIN,), "backward": (B.CHAIN, B.ISOLATED, B.FREE)}[kind]
    L.run(schedules[-1])
    L.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=L.stream_msg):
        L.run(schedules[-1])
    steps = [lambda d=L.desc(s): B.adaqp_layer_step(d) for s in schedules] + [graph.replay, lambda: L.run(B.CHAIN)]
    n, rng = p.n_rows, np.random.default_rng(6)
    ptr = np.arange(n + 1)
    for rowptr in (np.concatenate([[0], np.cumsum(rng.permutation(np.diff(p.rowptr)))]), np.clip(p.rowptr + 1, 0, p.nnz),
                   np.clip(p.rowptr - 3, 0, p.nnz), np.where(ptr > n // 2, p.nnz, 0), np.where(ptr > n - 2, p.nnz - 5, 5),
                   np.full(n + 1, p.nnz // 2), p.rowptr):
        rowptr = np.ascontiguousarray(rowptr, dtype=np.int64)
        L.rowptr.data.copy_(torch.from_numpy(rowptr))
        _, _, _, out64, mag = _oracle_layer(oracle, replace(p, rowptr=rowptr), 3)
        for step in steps:
            L.out.fill_(float("nan"))
            torch.cuda.synchronize()
            step()
            torch.cuda.synchronize()
            got = L.out.cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - out64) <= SPMM_RTOL * mag + 1e-30)


def test_layer_step_fused_receive_with_a_tiled_range(oracle):
    """The central rows tiled, the marginal ones read from the receive buffer: two streams, the same bits in every schedule,
    the halo rows of the feature matrix untouched."""
    p = make_partition(CONFIGS["c0"])
    cfg, seed = p.cfg, 1234
    _, _, _, out64, mag = _oracle_layer(oracle, p, seed)
    want = None
    for schedule in (B.SERIAL, B.ISOLATED, B.FREE, B.CHAIN, None):
        L = LayerStep(p, DEV, seed=seed, fused_receive=True, tiled=True)
        assert L.tile_off_overlap is not None and L.default_schedule() == B.ISOLATED
        d = L.desc(B.ISOLATED)
        assert d.tile_off_overlap_dev and not d.tile_off_dependent_dev and d.slot_of_row_dev
        L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        out = L.out.cpu().numpy()
        assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
        assert bool(torch.isnan(L.feat[cfg.n_local: cfg.n_local + cfg.n_send]).all())
        want = out if want is None else want
        assert np.array_equal(out.view(np.uint32), want.view(np.uint32)), f"schedule {schedule}"


@pytest.mark.parametrize("fused", [False, True])
def test_layer_step_with_a_range_of_unsorted_rows(oracle, fused):
    """Long rows whose range is tiled beside short ones that list their columns in no order, which tiles cannot take: the step of
    all rows, also after the receive that it was made for is switched."""
    _say(f"layer step, unsorted rows, fused {fused}")
    p = make_partition(replace(CONFIGS["c0"], n_local=24_000, n_halo=5_000, n_send=4_000, dim=256))
    b, e = p.dependent_rows
    rng = np.random.default_rng(11)
    long_rows = np.sort((np.arange(110) * 218 + rng.integers(0, 24_000, size=(b, 1))) % 24_000, axis=1)
    short_rows = np.stack([np.full(e - b, 28_000), np.arange(e - b), 24_000 + np.arange(e - b)], axis=1)
    col = np.concatenate([long_rows.reshape(-1), short_rows.reshape(-1)]).astype(np.int32)
    p = replace(p, rowptr=np.concatenate([[0], np.cumsum(np.repeat([110, 3], [b, e - b]))]).astype(np.int64), col=col,
                val=rng.standard_normal(col.size).astype(np.float32))
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    L = LayerStep(p, DEV, seed=9, fused_receive=fused)
    assert L.segments_overlap and L.tile_off_dependent is None
    for fused_now in (fused, not fused, fused):
        L.set_fused_receive(fused_now)
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run()
        L.synchronize()
        assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
    with pytest.raises(B.AdaqpError):                                  # tiles that are asked for are refused as ever
        LayerStep(p, DEV, seed=9, tiled=True)


@pytest.mark.parametrize("how", [dict(tiled=False), dict(fused_receive=True), dict(tiled=False, fused_receive=True)])
@pytest.mark.parametrize("twice", [False, True])
def test_layer_step_with_long_unsorted_rows(oracle, how, twice):
    """Long rows that list their columns in no order, or one of them twice: refused where they would have to be tiled, and nowhere else."""
    _say(f"layer step, long unsorted rows, {how} twice={twice}")
    p = make_partition(replace(CONFIGS["c0"], mean_degree=4000.0))
    b, e = p.dependent_rows if "tiled" not in how else (0, p.n_rows)
    assert p.rowptr[e] - p.rowptr[b] >= 128 * (e - b)
    col = p.col.copy()
    for r in range(b, e):
        row = col[p.rowptr[r]: p.rowptr[r + 1]]
        row[:] = row[::-1]
        if twice:
            row[1] = row[0]
    p = replace(p, col=col)
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    with pytest.raises(B.AdaqpError):
        LayerStep(p, DEV, seed=9)
    L = LayerStep(p, DEV, seed=9, **how)
    assert L.pieces_dependent
    L.run()
    L.synchronize()
    assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("which", ["feat", "out", "both"])
@pytest.mark.parametrize("ld,offset", [(128, 4), (129, 0), (160, 33)])
@pytest.mark.parametrize("fused", [False, True])
def test_layer_step_with_matrices_put_in_its_place(oracle, which, ld, offset, fused):
    """A step whose rows were planned in pieces, with matrices of its caller's that do not start on lines or have no whole lines."""
    _say(f"layer step, other matrices, {which} ld={ld} offset={offset} fused={fused}")
    p = make_partition(CONFIGS["c0"])
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    L = LayerStep(p, DEV, seed=9, fused_receive=fused)
    assert L.pieces_both and L.pieces_overlap
    for name in ("feat", "out") if which == "both" else (which,):
        n, dim = getattr(L, name).shape
        mine = torch.full((offset + n * ld,), float("nan"), device=DEV)[offset:].view(n, ld)[:, :dim]
        mine.copy_(getattr(L, name))
        setattr(L, name, mine)
    for schedule in (B.CHAIN, B.ISOLATED):
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("fused", [False, True])
def test_layer_step_with_a_taller_matrix_in_its_place(oracle, fused):
    """More rows of feat than the step was made with, none of them listed: tables of the rows there were are not written past their ends."""
    _say(f"layer step, taller feat, fused={fused}")
    p = make_partition(CONFIGS["c0"])
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    L = LayerStep(p, DEV, seed=9, fused_receive=fused)
    n, taller = L.feat.shape[0], torch.full((L.feat.shape[0] + 5_000, L.feat.stride(0)), float("nan"), device=DEV)
    taller[:n, :L.dim] = L.feat
    L.feat = taller[:, :L.dim]
    d = L.desc(B.CHAIN)
    assert d.n_feat_rows == n + 5_000 and not d.packed_row_dev
    L.run()
    L.synchronize()
    assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("status", [B.ESIZE, B.EINVAL])
@pytest.mark.parametrize("tiled", [False, True])
def test_layer_step_without_a_plan_of_pieces(oracle, monkeypatch, status, tiled):
    """A plan that the library refuses is done without: rows and segments are cut on the device."""
    _say(f"layer step, no plan of pieces, status {status} tiled={tiled}")
    p = make_partition(CONFIGS["c0"])

    def refuse(*args):
        raise B.AdaqpError(status, "plan")
    monkeypatch.setattr(B, "adaqp_plan_spmm_pieces", refuse)
    L = LayerStep(p, DEV, seed=9, tiled=tiled)
    assert bool(L.segments_overlap) == tiled and not L.segments_overlap.c.pieces.n_pieces and not L.pieces_overlap and not L.pieces_both
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    for schedule in (B.CHAIN, B.ISOLATED):
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


def test_layer_step_made_with_fused_receive_plans_tiles_when_it_is_switched_off(oracle):
    """Nothing reads tiles of received rows that stay packed: they are planned when these rows are to be de-quantised first."""
    _say("layer step, tiles after fused receive")
    p = make_partition(CONFIGS["c0"])
    _, _, _, out64, mag = _oracle_layer(oracle, p, 9)
    L = LayerStep(p, DEV, seed=9, fused_receive=True, tiled=True)
    assert L.segments_overlap and L.tile_off_dependent is None and not L.segments_dependent
    fused = L.desc(B.ISOLATED)
    L.set_fused_receive(False)
    assert L.tile_off_dependent is not None and L.segments_dependent
    for d in (L.desc(B.ISOLATED), fused, L.desc(B.CHAIN)):
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        B.adaqp_layer_step(d)
        L.synchronize()
        assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


def _c0_partition(name):
    if name == "c0":
        return make_partition(CONFIGS["c0"])
    return make_partition(replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))


@pytest.mark.parametrize("name", ["c0", "c0_backward"])
@pytest.mark.parametrize("schedule", [B.ISOLATED, B.FREE])
def test_layer_step_is_ordered_with_both_streams(name, schedule):
    """A step of any size: what the caller has queued on stream_agg comes before the overlapped aggregation, what it queues
    there afterwards comes after it, and synchronising stream_msg covers both."""
    p = _c0_partition(name)
    L = LayerStep(p, DEV, seed=5)
    L.run(B.SERIAL)
    L.synchronize()
    want = L.out.clone()
    (ob, oe), (db, de) = p.overlap_rows, p.dependent_rows
    x = torch.full((4096, 4096), 2.0 ** -12, device=DEV)
    y = torch.empty_like(x)

    def slow():
        for _ in range(10):
            torch.mm(x, x, out=y)

    slow()
    L.out.fill_(float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.stream(L.stream_agg):
        slow()
        L.out[ob:oe].fill_(5.0)
    L.run(schedule)
    L.stream_msg.synchronize()
    assert L.stream_agg.query()
    torch.cuda.synchronize()
    assert torch.equal(L.out.view(torch.int32), want.view(torch.int32))
    L.out.fill_(float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.stream(L.stream_msg):
        slow()
    L.run(schedule)
    with torch.cuda.stream(L.stream_agg):
        seen = L.out[ob:oe].clone()
    torch.cuda.synchronize()
    if not p.cfg.backward:                                  # backward: received gradients are added on stream_msg
        assert torch.equal(seen.view(torch.int32), want[ob:oe].view(torch.int32))
    else:
        assert not bool(torch.isnan(seen).any())
    assert torch.equal(L.out.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("name", ["c0", "c0_backward"])
@pytest.mark.parametrize("fused", [False, True])
def test_layer_step_chain(oracle, name, fused):
    """CHAIN, which a step without a schedule takes here: one aggregation launch for both ranges against the oracle; with the
    received rows still packed the same bits; the bits of SERIAL where the ranges do not touch or no workspace holds both."""
    p = _c0_partition(name)
    cfg, seed = p.cfg, 1234
    _, _, _, out64, mag = _oracle_layer(oracle, p, seed)

    def step(schedule, **kw):
        L = LayerStep(p, DEV, seed=seed, fused_receive=fused, **kw)
        if not cfg.backward:
            L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        return L, L.desc(schedule)

    L, d = step(B.CHAIN, backward_receive=False)
    assert L.default_schedule() == B.CHAIN
    B.adaqp_layer_step(d)
    L.synchronize()
    out = L.out.cpu().numpy()
    assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
    again, _ = step(B.CHAIN, backward_receive=False)
    again.set_fused_receive(False)
    again.run()
    again.synchronize()
    assert np.array_equal(again.out.cpu().numpy().view(np.uint32), out.view(np.uint32))
    assert torch.equal(again.recv_packed, L.recv_packed)
    # what keeps the ranges apart: no room for both, a row between them; received gradients are added in either case
    bits = {}
    for cut in ("small", "gap"):
        for schedule in (B.SERIAL, B.CHAIN, B.ISOLATED):
            L, d = step(schedule)
            if cut == "small":
                d.workspace_overlap_bytes = B.adaqp_spmm_workspace_bytes(d.overlap_end - d.overlap_begin, d.overlap_nnz, cfg.dim)
                d.workspace_dependent_bytes = B.adaqp_spmm_workspace_bytes(d.dependent_end - d.dependent_begin,
                                                                           d.dependent_nnz, cfg.dim)
            else:
                d.overlap_end -= 1
                d.overlap_nnz = int(p.rowptr[d.overlap_end] - p.rowptr[d.overlap_begin])
                L.out[d.overlap_end].fill_(3.0)
                torch.cuda.synchronize()
            B.adaqp_layer_step(d)
            L.synchronize()
            bits.setdefault(cut, []).append(L.out.view(torch.int32).clone())
        assert torch.equal(bits[cut][0], bits[cut][1]) and torch.equal(bits[cut][0], bits[cut][2]), cut
        assert not bool(torch.isnan(bits[cut][0].view(torch.float32)).any())


@pytest.mark.parametrize("extra,offset", [(0, 0), (5, 4), (7, 1), ((1 << 28) + 3, 1), ((1 << 32) + 77, 1)])
def test_layer_step_copies_the_whole_buffer(extra, offset):
    """The loop-back of a send buffer of any size and alignment: units of 16, 4 and 1 bytes, what they leave over, and more of
    them than a launch has threads (a backward step without receive reads nothing of the copy)."""
    p = _c0_partition("c0_backward")
    L = LayerStep(p, DEV, seed=5, backward_receive=False)
    n = L.plan.packed_bytes + extra
    _say(f"loop-back {n} bytes at offset {offset}")
    sent = torch.randint(0, 256, (n,), dtype=torch.uint8, device=DEV)
    received = torch.full((n + 32,), 7, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    d = L.desc(B.SERIAL)
    d.packed_dev, d.packed_bytes, d.recv_packed_dev = sent.data_ptr(), n, received.data_ptr() + offset
    B.adaqp_layer_step(d)
    L.synchronize()
    assert torch.equal(received[offset:offset + n], sent)
    assert bool((received[:offset] == 7).all()) and bool((received[offset + n:] == 7).all())
    assert torch.equal(L.recv_params, L.params)


@pytest.mark.parametrize("kind,dim,extra,offset", [("forward", 128, 0, 0), ("forward", 97, 5, 4), ("forward", 2100, 3, 16), ("fused", 66, 0, 0),
                                                   ("fused", 130, 4099, 8), ("backward", 128, 0, 0), ("backward", 97, 5, 4), ("backward", 2100, 3, 16)])
def test_layer_step_chain_copies_beside_the_receive(kind, dim, extra, offset):
    """CHAIN receives from where the loop-back copy takes the bytes, and copies in the same launch: what the other schedules leave, in every
    buffer, also bytes that no message covers and messages that are skipped."""
    _say(f"chain, {kind} dim={dim} extra={extra} offset={offset}")
    backward = kind == "backward"
    p = make_partition(replace(CONFIGS["c0"], dim=dim) if not backward else
                       replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=dim))
    left = []
    for schedule in (B.SERIAL, B.CHAIN):
        L = LayerStep(p, DEV, seed=5, fused_receive=kind == "fused")
        n = L.plan.packed_bytes + extra
        sent = torch.full((n + 16,), 3, dtype=torch.uint8, device=DEV)
        received = torch.full((n + 48,), 7, dtype=torch.uint8, device=DEV)
        L.params.fill_(0.5)
        L.plan.bits[3], L.plan.send_idx[7] = 5, -1                          # skipped: their bytes and (Z, S) stay what they are
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        d = L.desc(schedule)
        d.packed_dev, d.packed_bytes, d.recv_packed_dev = sent.data_ptr(), n, received.data_ptr() + offset
        if backward:
            d.overlap_end -= 1                                              # what is sent are sums: two launches in either schedule, the same bits
        B.adaqp_layer_step(d)
        L.synchronize()
        assert torch.equal(received[offset:offset + n], sent[:n]) and torch.equal(L.recv_params, L.params)
        assert bool((received[:offset] == 7).all()) and bool((received[offset + n:] == 7).all())
        left.append([t.contiguous().view(torch.int32).clone() for t in (L.out, L.feat, L.params, L.beta)] + [sent])
    for a, b in zip(left[0][not backward:], left[1][not backward:]):
        assert torch.equal(a, b)
    if not backward:                                                        # rows in one launch may be cut in other places
        a, b = (x[0].view(torch.float32).double() for x in left)
        assert not bool(torch.isnan(b).any()) and float((a - b).norm()) <= 1e-6 * float(a.norm())


@pytest.mark.parametrize("kind,where", [("forward", "feat"), ("forward", "out"), ("fused", "out"), ("fused", "workspace"), ("backward", "workspace")])
def test_layer_step_chain_with_send_buffers_in_memory_that_is_used_again(kind, where):
    """Nothing reads the send buffers once the messages are copied: they may lie in rows of feat that are received, in out or in a workspace."""
    _say(f"chain, {kind}, send buffers in {where}")
    p = make_partition(replace(CONFIGS["c0"], n_local=6_000, n_halo=900, n_send=900, mean_degree=60.0, dim=70) if kind != "backward" else
                       replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))
    left = []
    for shared in (False, True):
        L = LayerStep(p, DEV, seed=5, fused_receive=kind == "fused")
        d = L.desc(B.CHAIN)
        assert d.pieces_both.n_pieces > 0
        if shared:
            received = np.sort(p.halo_idx)
            assert kind == "backward" or np.array_equal(received, np.arange(p.n_rows, p.n_rows + received.size))
            memory = {"feat": L.feat[p.n_rows if kind != "backward" else 0:], "out": L.out, "workspace": L.ws_overlap}[where]
            assert d.workspace_overlap_bytes >= d.workspace_dependent_bytes
            room = memory.numel() * memory.element_size()
            params_at = -(-d.packed_bytes // 256) * 256
            assert params_at + 8 * d.n_send <= room
            d.packed_dev = memory.data_ptr()
            d.params_dev = memory.data_ptr() + params_at
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        B.adaqp_layer_step(d)
        L.synchronize()
        left.append([t.contiguous().view(torch.int32).clone() for t in (L.out, L.feat, L.recv_params, L.beta)] + [L.recv_packed.clone()])
    for a, b in zip(*left):
        assert torch.equal(a, b)


def _launches(L, d):
    """Kernels of one step, counted in a capture that is not replayed."""
    hip = ctypes.CDLL("libamdhip64.so")
    graph, nodes = ctypes.c_void_p(), ctypes.c_size_t(0)
    stream = ctypes.c_void_p(L.stream_msg.cuda_stream)
    assert hip.hipStreamBeginCapture(stream, ctypes.c_int(2)) == 0
    B.adaqp_layer_step(d)
    assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return nodes.value


@pytest.mark.parametrize("kind", ["forward", "fused", "backward"])
def test_layer_step_chain_has_no_launch_for_the_copy(kind):
    """One launch fewer than where the send buffers lie in memory that the receive writes, whose copy is a launch of its own."""
    _say(f"launches of a chain, {kind}")
    p = make_partition(replace(CONFIGS["c0"], n_local=6_000, n_halo=900, n_send=900, mean_degree=60.0, dim=66) if kind != "backward" else
                       replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))
    L = LayerStep(p, DEV, seed=5, fused_receive=kind == "fused")
    d = L.desc(B.CHAIN)
    assert d.pieces_both.n_pieces > 0 and bool(d.slot_of_row_dev) == (kind == "fused")
    L.run(B.CHAIN)
    L.synchronize()
    beside = _launches(L, d)
    d.packed_dev = L.out.data_ptr()
    assert _launches(L, d) == beside + 1
    sums = int(d.pieces_both.n_sums > 0)
    assert beside == (2 if kind == "fused" else 3) + sums


def test_layer_step_packed_rows_in_slices_of_two_lines(oracle, monkeypatch):
    """Seven lines, a plan of two per slice, long pieces of rows shorter than 100 entries: packed rows are walked two lines at a time, the last
    slice one.  Against the oracle, and the bits of the step that reads what was received from feat."""
    _say("layer step, packed rows in slices of two lines")
    monkeypatch.setattr(B, "adaqp_spmm_pieces_rule", lambda *args, **options: (2, -np.inf))
    p, want = make_partition(replace(CONFIGS["c0"], n_local=24_000, n_halo=6_000, n_send=4_800, mean_degree=40.0, dim=220)), None
    _, _, _, out64, mag = _oracle_layer(oracle, p, 5)
    for fused in (True, False):
        L = LayerStep(p, DEV, seed=5, tiled=False, fused_receive=fused)
        c = L.pieces_both.c
        assert (c.entries, c.lines_per_slice) == (768, 2) and p.nnz < 100 * c.n_seg
        L.run(B.CHAIN)
        L.synchronize()
        got = L.out.cpu().numpy()
        assert np.all(np.abs(got.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
        want = got if want is None else want
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


def test_mean_aggregator_layer_step(oracle):
    """GraphSAGE-style mean coefficients (1 / row degree) through the same step."""
    p = make_partition(replace(CONFIGS["c0"], aggregator="mean"))
    _, _, feat_w, out64, mag = _oracle_layer(oracle, p, 9)
    L = LayerStep(p, DEV, seed=9)
    L.out.fill_(float("nan"))
    L.run(B.ISOLATED)
    L.synchronize()
    out = L.out.cpu().numpy()
    assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)
    assert np.array_equal(L.feat.cpu().numpy().view(np.uint32), feat_w.view(np.uint32))
    # a mean of values stays inside their range
    lo, hi = feat_w.min(), feat_w.max()
    assert out.min() >= lo - 1e-4 and out.max() <= hi + 1e-4


def test_trace_assign_replan_loop(oracle):
    """One period of Sec. 3.3: the step traces beta, the assigner turns it into widths, the next step runs with
    the new layout.  The oracle does the same from its own trace; widths and bytes must agree exactly."""
    import dataclasses
    from oracle import assigner as A
    p = make_partition(CONFIGS["c0"])
    cfg = p.cfg
    seed = 77
    L = LayerStep(p, DEV, seed=seed)
    L.run(B.SERIAL)
    L.synchronize()
    pl = L.plan
    beta_gpu = L.beta.cpu().numpy()
    peer_sorted = np.ascontiguousarray(p.peer_of_slot[pl.perm])
    theta = np.array([1.0, 1.5, 0.7]) * 1e-8
    gamma = np.full(cfg.n_peers, 1e-5)
    lam, group = 1e-7, 20
    bits_sorted, obj = B.adaqp_assign_bits(beta_gpu, peer_sorted, cfg.n_peers, cfg.dim, group, lam, theta, gamma)
    beta_cpu = oracle.trace_beta(p.feat, cfg.dim, pl.send_idx_host, L.alpha_sq_host)
    want_bits = A.greedy(beta_cpu, peer_sorted, cfg.n_peers, cfg.dim, group, lam, theta, gamma)
    assert np.array_equal(bits_sorted, want_bits)
    assert set(np.unique(bits_sorted)) == {2, 4, 8}
    f, _, _ = A.objective(beta_cpu, peer_sorted, cfg.n_peers, cfg.dim, bits_sorted, lam, theta, gamma)
    assert obj[0] == pytest.approx(f, rel=1e-12)
    # the assignment beats the one it replaces on the objective it was chosen for
    f_old, _, _ = A.objective(beta_cpu, peer_sorted, cfg.n_peers, cfg.dim, pl.bits_host, lam, theta, gamma)
    assert f < f_old
    bits_new = np.zeros_like(p.bits)
    bits_new[pl.perm] = bits_sorted                                  # back to the caller's slot order
    p2 = dataclasses.replace(p, bits=bits_new)
    packed_w, params_w, feat_w, out64, mag = _oracle_layer(oracle, p2, seed)
    L2 = LayerStep(p2, DEV, seed=seed)
    L2.run(B.ISOLATED)
    L2.synchronize()
    assert np.array_equal(L2.recv_packed.cpu().numpy()[: L2.plan.packed_bytes], packed_w)
    assert np.array_equal(L2.feat.cpu().numpy().view(np.uint32), feat_w.view(np.uint32))
    assert np.all(np.abs(L2.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("name", ["c0", "c0_backward"])
def test_layer_step_with_tiled_aggregation(oracle, name):
    """Both row ranges through the L2-tiled kernel, every schedule, forward and backward."""
    if name == "c0":
        p = make_partition(CONFIGS["c0"])
    else:
        p = make_partition(replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))
    cfg = p.cfg
    seed = 4321
    packed_w, params_w, feat_w, out64, mag = _oracle_layer(oracle, p, seed)
    first = None
    for schedule in (B.SERIAL, B.ISOLATED, B.FREE):
        L = LayerStep(p, DEV, seed=seed, tiled=True, backward_receive=False)
        assert L.tile_off_overlap is not None and L.tile_off_dependent is not None
        if not cfg.backward:
            L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        out = L.out.cpu().numpy()
        assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30), f"schedule {schedule}"
        if not cfg.backward:
            assert np.array_equal(L.recv_packed.cpu().numpy()[: L.plan.packed_bytes], packed_w)
            assert np.array_equal(L.feat.cpu().numpy().view(np.uint32), feat_w.view(np.uint32))
        if first is None:
            first = out
        assert np.array_equal(out.view(np.uint32), first.view(np.uint32)), "schedules disagree"


@pytest.mark.parametrize("name", ["c0", "c0_backward"])
def test_layer_step_with_panels(oracle, name):
    """Tiled aggregation with the longer rows of both ranges in dense panels, every schedule, both directions."""
    if name == "c0":
        p = make_partition(CONFIGS["c0"])
    else:
        p = make_partition(replace(CONFIGS["c4"], n_local=2000, n_halo=1800, n_send=1500, mean_degree=9.0, dim=128))
    cfg = p.cfg
    seed = 8765
    deg = np.diff(p.rowptr)
    min_row = max(int(np.quantile(deg[deg > 0], 0.9)), 2)               # the longest tenth of the rows
    packed_w, params_w, feat_w, out64, mag = _oracle_layer(oracle, p, seed)
    first = None
    for schedule in (B.SERIAL, B.ISOLATED, B.FREE):
        L = LayerStep(p, DEV, seed=seed, tiled=True, panels=True, backward_receive=False, panel_min_row=min_row)
        assert L.panels_overlap and L.panels_dependent
        n_taken = int(np.count_nonzero(L.panels_overlap.tensors["panel_rows"].cpu().numpy() >= 0)) + \
            int(np.count_nonzero(L.panels_dependent.tensors["panel_rows"].cpu().numpy() >= 0))
        ob, oe = p.overlap_rows
        db, de = p.dependent_rows
        assert n_taken == int(np.count_nonzero(deg[ob:oe] >= min_row)) + int(np.count_nonzero(deg[db:de] >= min_row))
        if not cfg.backward:
            L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.out.fill_(float("nan"))
        torch.cuda.synchronize()
        L.run(schedule)
        L.synchronize()
        out = L.out.cpu().numpy()
        assert np.all(np.abs(out.astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30), f"schedule {schedule}"
        if not cfg.backward:
            assert np.array_equal(L.recv_packed.cpu().numpy()[: L.plan.packed_bytes], packed_w)
            assert np.array_equal(L.feat.cpu().numpy().view(np.uint32), feat_w.view(np.uint32))
        if first is None:
            first = out
        assert np.array_equal(out.view(np.uint32), first.view(np.uint32)), "schedules disagree"
    # without panels the same rows come out of the tiled kernel: same sums up to rounding order
    L = LayerStep(p, DEV, seed=seed, tiled=True, backward_receive=False, panels=False)
    assert not L.panels_overlap and not L.panels_dependent
    L.run(B.SERIAL)
    L.synchronize()
    assert np.all(np.abs(L.out.cpu().numpy().astype(np.float64) - out64) <= SPMM_RTOL * mag + 1e-30)


@pytest.mark.parametrize("schedule_name", ["serial", "isolated", "free", "chain", "isolated_tiled_panels", "free_tiled_panels"])
def test_layer_step_captured_in_a_graph(schedule_name):
    """The step allocates nothing and clears nothing with memset, so it can be captured into a HIP graph; every
    replay (with eager work and synchronisations in between) must give the bits of the eager step.  With tiles
    and panels in both row ranges the two streams wait for each other twice more (the panel kernels run beside
    the tiled ones)."""
    schedule = {"serial": B.SERIAL, "isolated": B.ISOLATED, "free": B.FREE, "chain": B.CHAIN}[schedule_name.split("_")[0]]
    p = make_partition(CONFIGS["c0"])
    cfg = p.cfg
    if schedule_name.endswith("tiled_panels"):
        deg = np.diff(p.rowptr)
        L = LayerStep(p, DEV, seed=99, tiled=True, panels=True,
                      panel_min_row=max(int(np.quantile(deg[deg > 0], 0.9)), 2))
        assert L.panels_overlap and L.panels_dependent
    else:
        L = LayerStep(p, DEV, seed=99)
    L.run(schedule)
    L.synchronize()
    want_out = L.out.clone()
    want_feat = L.feat.clone()
    want_packed = L.recv_packed.clone()
    desc = L.desc(schedule)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=L.stream_msg):
        B.adaqp_layer_step(desc)
    for replay in range(3):
        L.out.fill_(float("nan"))                                   # eager work between the replays
        L.feat[cfg.n_local: cfg.n_local + cfg.n_send] = float("nan")
        L.recv_packed.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.recv_packed, want_packed), f"replay {replay}: packed bytes"
        assert torch.equal(L.feat.view(torch.int32), want_feat.view(torch.int32)), f"replay {replay}: halo rows"
        assert torch.equal(L.out.view(torch.int32), want_out.view(torch.int32)), f"replay {replay}: aggregate"
