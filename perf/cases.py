"""The work a user of this package has it do, as cases to be timed: layer steps of whole partitions (forward,
backward, both with and without the options of LayerStep), the individual calls for callers that own the exchange,
and the periodic re-assignment of bit-widths.

A case is a dict of plain values.  `prepare` draws a partition on the GPU (same laws as synth.py: Zipf or log-normal
row degrees, power-law column popularity, GCN coefficients, an unbalanced split over peers) and makes what a training
program keeps between steps: the LayerStep, or the index arrays, plans and buffers of the individual calls.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2306_01381_amd import binding as B
from paper_2306_01381_amd.layer import LayerStep, SendPlan
from paper_2306_01381_amd.synth import Partition, PartitionConfig

DEV = "cuda:0"


def _step(name, rows, halo, edges, dim, send, peers, feat, bits, backward=False, receive=True, law="zipf",
          fused=False):
    return dict(name=name, kind="step", rows=rows, halo=halo, edges=edges, dim=dim, send=send, peers=peers, feat=feat,
                bits=bits, backward=backward, receive=receive, law=law, fused=fused)


def listed():
    return [
        # Forward layer steps.  The smallest partition in use: a step of a few microseconds of work, so launches, copies
        # and the host path are what a training loop over a small graph waits for.
        _step("forward tiny", 2_000, 600, 20_656, 128, 400, 3, "normal", "uniform"),
        # One of four parts of a mid-size graph, a narrow hidden layer whose width fills no vector evenly; received rows are
        # aggregated straight from the receive buffer.
        _step("forward fused ragged", 24_000, 10_000, 420_000, 66, 9_000, 3, "relu", "mix", fused=True),
        # One of four parts of a 233K-node / 114M-edge graph with 602 input features: thousands of entries in the longest rows.
        _step("forward dense 602", 58_000, 40_000, 28_240_000, 602, 30_000, 3, "normal", "mix"),
        # The same sizes in a hidden layer, with row degrees of a milder skew.
        _step("forward dense hidden", 58_000, 40_000, 27_790_000, 256, 30_000, 3, "relu", "mix", law="lognormal"),
        # One of eight parts of a 2.45M-node / 62M-edge graph, hidden layer, everything sent at two bits.
        _step("forward sparse hidden", 306_000, 150_000, 7_680_000, 256, 120_000, 7, "relu", "all2"),
        # One of four parts of a 716K-node / 7M-edge graph, 300 input features with heavy tails.
        _step("forward sparse 300", 179_000, 90_000, 1_963_000, 300, 80_000, 3, "heavy_tail", "uniform"),
        # Backward layer steps: one of eight parts of a 1.57M-node / 132M-edge graph, widths as the assigner gives them.
        _step("backward large", 196_000, 180_000, 16_250_000, 256, 150_000, 7, "grad", "adaptive", backward=True,
              receive=False),
        # A part of a denser, smaller graph; every message at eight bits, what the peers send back is added.
        _step("backward dense 8 bit", 30_000, 20_000, 4_000_000, 128, 16_000, 3, "grad", "all8", backward=True),
        # A caller that owns the exchange and whose matrices have no padding: send, receive and aggregation as single calls.
        dict(name="calls unpadded odd", kind="calls", rows=60_000, halo=30_000, edges=1_000_000, dim=301, send=25_000,
             peers=5, feat="normal", bits="uniform", law="zipf", pad=False),
        # The message path by itself, as a trainer with its own aggregation uses it.
        dict(name="messages forward", kind="messages", rows=200_000, halo=160_000, dim=256, send=150_000, peers=7,
             feat="normal", bits="adaptive", pad=True),
        # Gradients that came back from the peers, added to the rows of their owners.
        dict(name="messages backward", kind="gradients", rows=196_000, dim=256, send=150_000, peers=7, bits="adaptive",
             pad=True),
        # Once per period: widths from the traced betas, and the send plan rebuilt for them.
        dict(name="reassign", kind="reassign", rows=200_000, dim=256, send=100_000, peers=7, group=100),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 10 + ["backward"] * 4 + ["calls"] * 2 + ["messages"] * 2 + ["gradients", "reassign"])
    dim = rng.choice([_log_uniform(rng, 16, 602), _log_uniform(rng, 4, 75) * 8])
    bits = rng.choice(["uniform", "mix", "all2", "adaptive", "all8"])
    peers = rng.randint(1, 7)
    if kind in ("messages", "gradients", "reassign"):
        rows = _log_uniform(rng, 2_000, 200_000)
        send = max(peers, int(rows * rng.uniform(0.2, 0.7)))
        if kind == "reassign":
            return dict(kind=kind, rows=rows, dim=dim, send=min(send, 100_000), peers=peers, group=rng.choice([20, 50, 100, 300]))
        pad = rng.random() < 0.75
        while send * dim > 150_000 * 256:
            send //= 2
        if kind == "gradients":
            return dict(kind=kind, rows=rows, dim=dim, send=send, peers=peers, bits=bits, pad=pad)
        return dict(kind=kind, rows=rows, halo=send + rng.randint(0, rows // 4), dim=dim, send=send, peers=peers,
                    feat=rng.choice(["normal", "relu", "heavy_tail"]), bits=bits, pad=pad)
    while True:
        rows = _log_uniform(rng, 2_000, 306_000)
        edges = int(rows * math.exp(rng.uniform(math.log(4), math.log(500))))
        # no more entries, products or rows than the largest listed cases
        if edges <= 28_000_000 and edges * dim <= 17_000_000_000 and rows * dim <= 80_000_000:
            break
    halo = max(8, int(rows * rng.uniform(0.25, 0.9)))
    send = max(peers, int(min(halo, rows) * rng.uniform(0.5, 0.9)))
    law = rng.choice(["zipf", "zipf", "lognormal"])
    feat = rng.choice(["normal", "relu", "heavy_tail"])
    if kind == "calls":
        return dict(kind=kind, rows=rows, halo=halo, edges=edges, dim=dim, send=send, peers=peers, feat=feat, bits=bits,
                    law=law, pad=rng.random() < 0.5)
    backward = kind == "backward"
    c = _step("", rows, halo, edges, dim, send, peers, "grad" if backward else feat, bits, backward,
              not backward or bits == "all8", law, not backward and rng.random() < 0.2)
    del c["name"]
    return c


# ---- inputs ----------------------------------------------------------------------------------------------------------

def _degree_weights(g, n, mean, cap, law):
    if law == "zipf":                                   # Zipf(1.5), clipped
        k = torch.arange(1, 13_000, dtype=torch.float64, device=DEV)
        cdf = torch.cumsum(k ** -1.5 / 2.6123753486854883, 0)
        raw = torch.searchsorted(cdf, torch.rand(n, generator=g, dtype=torch.float64, device=DEV)).double() + 1
    else:                                               # log-normal, sigma 1
        raw = torch.randn(n, generator=g, dtype=torch.float64, device=DEV).exp()
    return (raw * (mean / raw.mean())).clamp(1, cap)


def _popularity(g, n):
    cdf = torch.cumsum(torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** -0.6, 0)
    cdf /= cdf[-1].clone()
    perm = torch.randperm(n, generator=g, device=DEV)
    return lambda u: perm[torch.searchsorted(cdf, u).clamp_(max=n - 1)]


def _graph(g, case):
    """rowptr, col, val of the partition's graph (rows = local nodes, columns = local + halo nodes; rows without remote
    neighbours first), with exactly case["edges"] entries unless the rows cannot hold that many."""
    n, halo, want = case["rows"], case["halo"], case["edges"]
    n_cols, n_central = n + halo, n - min(n, case["send"])
    rows = torch.arange(n, device=DEV)
    marg = rows[n_central:]
    draw_local, draw_halo = _popularity(g, n), _popularity(g, halo)
    share = torch.zeros(n, dtype=torch.float64, device=DEV)
    share[n_central:] = torch.rand(marg.numel(), generator=g, dtype=torch.float64, device=DEV) * 0.3 + 0.3
    deg = _degree_weights(g, n, want / n, max(1, n // 2), case["law"])
    # a self-loop in every row and a remote neighbour in every marginal one
    fixed = torch.unique(torch.cat([rows * n_cols + rows, marg * n_cols + n + draw_halo(
        torch.rand(marg.numel(), generator=g, dtype=torch.float64, device=DEV))]))
    key = fixed
    for _ in range(6):
        short = want - key.numel()
        if short <= 0:
            break
        r = torch.repeat_interleave(rows, (deg * (1.25 * short / deg.sum())).ceil().long())
        u = torch.rand(r.numel(), generator=g, dtype=torch.float64, device=DEV)
        remote = torch.rand(r.numel(), generator=g, dtype=torch.float64, device=DEV) < share[r]
        key = torch.unique(torch.cat([key, r * n_cols + torch.where(remote, n + draw_halo(u), draw_local(u))]))
    if key.numel() > want:                              # drop the surplus at random, never the fixed entries
        rank = torch.rand(key.numel(), generator=g, device=DEV)
        rank[torch.searchsorted(key, fixed)] = -1.0
        key = key[torch.sort(torch.argsort(rank)[:want]).values]
    r, col = torch.div(key, n_cols, rounding_mode="floor"), key % n_cols
    d_row = torch.bincount(r, minlength=n).double()
    d_col = torch.cat([d_row, 1.0 + torch.bincount(col, minlength=n_cols)[n:].double()])
    val = (d_row[r] * d_col[col]).rsqrt().float()
    return r, col, val, n_central


def _rowptr(r, n):
    out = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    out[1:] = torch.cumsum(torch.bincount(r, minlength=n), 0)
    return out


def _features(g, kind, n, dim):
    x = torch.randn(n, dim, generator=g, device=DEV)
    if kind == "relu":
        return x.clamp_(min=0.0)
    if kind == "grad":
        return x.mul_(1e-3)
    if kind == "heavy_tail":                            # 50 columns of Student's t with three degrees of freedom
        c = torch.randperm(dim, generator=g, device=DEV)[:50]
        chi = torch.randn(n, c.numel(), 3, generator=g, device=DEV).square().sum(2)
        x[:, c] = x[:, c] / (chi / 3).sqrt()
    return x


def _peer_of_slot(n, peers):
    w = 1.0 / np.arange(1, peers + 1)
    cnt = np.maximum(1, np.floor(n * w / w.sum()).astype(np.int64))
    cnt[0] += n - cnt.sum()
    return np.repeat(np.arange(peers, dtype=np.int32), cnt)


def _bits(g, kind, n, score=None):
    if kind == "all2" or kind == "all8":
        return np.full(n, 2 if kind == "all2" else 8, dtype=np.uint8)
    # the shares of the widths are exact; "adaptive" gives the widest codes to the largest variance proxies
    key = -score if kind == "adaptive" and score is not None else torch.rand(n, generator=g, device=DEV)
    u = torch.argsort(torch.argsort(key)).double() / n
    eight, four = {"uniform": (1 / 3, 2 / 3), "mix": (0.1, 0.7), "adaptive": (0.15, 0.6)}[kind]
    b = torch.where(u < eight, 8, torch.where(u < four, 4, 2))
    return b.to(torch.uint8).cpu().numpy()


def _np(t, dtype):
    return t.to(dtype).cpu().numpy()


_streams = None


def _step_streams():
    """The one pair of streams all steps of a program run on."""
    global _streams
    if _streams is None:
        _streams = (torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV))
    return _streams


def _partition(g, case, seed):
    n, halo, send, peers = case["rows"], case["halo"], case["send"], case["peers"]
    r, col, val, n_central = _graph(g, case)
    cfg = PartitionConfig("case", n, halo, case["edges"] / n, case["dim"], send, peers, case["feat"], case["bits"],
                          backward=case["backward"], seed=seed)
    peer = _peer_of_slot(send, peers)
    if not case["backward"]:
        sent = n_central + torch.randperm(n - n_central, generator=g, device=DEV)[:send]
        return Partition(cfg, _np(_rowptr(r, n), torch.int64), _np(col, torch.int32), val.cpu().numpy(), n, n + halo,
                         (0, n_central), (n_central, n), n_central,
                         _features(g, case["feat"], n + halo, case["dim"]).cpu().numpy(), _np(sent, torch.int32), peer,
                         _bits(g, case["bits"], send), (n + np.arange(send)).astype(np.int32))
    # the transposed graph: rows = local + halo nodes, columns = local nodes; the halo rows are what is sent
    order = torch.sort(col * n + r).indices
    r, col, val = col[order], r[order], val[order]
    sent = n + torch.randperm(halo, generator=g, device=DEV)[:send]
    score = torch.zeros(n + halo, dtype=torch.float64, device=DEV).index_add_(0, r, val.double().square())
    back = torch.cat([n_central + torch.randperm(n - n_central, generator=g, device=DEV)[:int(c)]
                      for c in np.bincount(peer, minlength=peers)])
    return Partition(cfg, _np(_rowptr(r, n + halo), torch.int64), _np(col, torch.int32), val.cpu().numpy(), n + halo, n,
                     (0, n), (n, n + halo), n_central, _features(g, case["feat"], n, case["dim"]).cpu().numpy(),
                     _np(sent, torch.int32), peer, _bits(g, case["bits"], send, score[sent]), _np(back, torch.int32))


def _matrix(x, pad):
    if not pad:
        return x
    n, dim = x.shape
    out = torch.zeros(n, (dim + 31) // 32 * 32, device=DEV)[:, :dim]
    return out.copy_(x)


def _buffers(plan):
    return (torch.zeros(max(plan.packed_bytes, 4), dtype=torch.uint8, device=DEV),
            torch.zeros(plan.n, 2, dtype=torch.float32, device=DEV))


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind, dim, rows, send, peers = case["kind"], case["dim"], case["rows"], case["send"], case["peers"]
    s = dict(case=case, seed=seed)
    if kind == "step":
        s["step"] = LayerStep(_partition(g, case, seed), DEV, seed=seed, backward_receive=case["receive"],
                              fused_receive=case["fused"], streams=_step_streams())
        return s
    peer = _peer_of_slot(send, peers)
    sent = _np(torch.randperm(rows, generator=g, device=DEV)[:send], torch.int32)
    if kind == "reassign":
        var = torch.randn(send, generator=g, device=DEV).exp() * 1e-2
        s.update(beta=var.cpu().numpy(), peer=peer, sent=sent, halo=(rows + np.arange(send)).astype(np.int32),
                 theta=np.linspace(1.0, 2.0, peers) * 1e-8, gamma=np.full(peers, 1e-5))
        return s
    bits = _bits(g, case["bits"], send)
    if kind == "gradients":
        # each peer names a row at most once; different peers may name the same row
        back = torch.cat([torch.randperm(rows, generator=g, device=DEV)[:int(c)] for c in np.bincount(peer, minlength=peers)])
        plan = SendPlan(dim, sent, bits, peer, peers, _np(back, torch.int32), DEV, add_segments=True)
        grad, theirs = _features(g, "grad", rows, dim), _features(g, "grad", rows, dim)
        packed, params = _buffers(plan)
        B.adaqp_quantize_pack(theirs, dim, plan.send_idx, plan.bits, plan.row_offset, seed, packed, params)
        s.update(plan=plan, grad=_matrix(grad, case["pad"]), packed=packed, params=params)
        return s
    halo = case["halo"]
    if kind == "calls":
        r, col, val, n_central = _graph(g, case)
        s.update(rowptr=_rowptr(r, rows), col=col.int(), val=val)
        sent = _np(n_central + torch.randperm(rows - n_central, generator=g, device=DEV)[:send], torch.int32)
        s["out"] = _matrix(torch.zeros(rows, dim, device=DEV), case["pad"])
        s["workspace"] = torch.empty(max(256, B.adaqp_spmm_workspace_bytes(rows, col.numel(), dim)), dtype=torch.uint8,
                                     device=DEV)
    s["plan"] = SendPlan(dim, sent, bits, peer, peers, (rows + np.arange(send)).astype(np.int32), DEV)
    s["feat"] = _matrix(_features(g, case["feat"], rows + halo, dim), case["pad"])
    s["packed"], s["params"] = _buffers(s["plan"])
    s["alpha_sq"] = torch.rand(send, generator=g, device=DEV)
    s["beta"] = torch.zeros(send, device=DEV)
    return s


# ---- one pass --------------------------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind, dim = case["kind"], case["dim"]
    if kind == "step":
        L = s["step"]
        L.run()
        received = L.feat[case["rows"]:case["rows"] + case["send"]]
        if case["backward"]:
            return L.out, L.recv_packed, L.recv_params, L.beta
        if case["fused"]:
            return L.out, L.recv_packed, L.recv_params, L.beta
        return L.out, received, L.recv_packed, L.recv_params, L.beta
    if kind == "reassign":
        bits, objective = B.adaqp_assign_bits(s["beta"], s["peer"], case["peers"], dim, case["group"], 1e-7, s["theta"],
                                              s["gamma"])
        plan = SendPlan(dim, s["sent"], bits, s["peer"], case["peers"], s["halo"], DEV)
        return bits, objective, plan.send_idx, plan.bits, plan.row_offset, plan.halo_idx, plan.peer_byte_ptr
    p = s["plan"]
    if kind == "gradients":
        B.adaqp_unpack_dequant_add(s["packed"], s["params"], p.bits, p.row_offset, p.halo_idx, p.seg_order, p.seg_ptr, dim,
                                   s["grad"])
        return s["grad"]
    B.adaqp_quantize_pack_trace(s["feat"], dim, p.send_idx, p.bits, p.row_offset, s["seed"], s["packed"], s["params"],
                                s["alpha_sq"], s["beta"])
    B.adaqp_unpack_dequant(s["packed"], s["params"], p.bits, p.row_offset, p.halo_idx, dim, s["feat"])
    received = s["feat"][case["rows"]:case["rows"] + case["send"]]
    if kind == "messages":
        return received, s["packed"], s["params"], s["beta"]
    B.adaqp_spmm_csr(s["rowptr"], s["col"], s["val"], 0, case["rows"], s["feat"], dim, s["out"], s["workspace"])
    return s["out"], received, s["packed"], s["params"], s["beta"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

_MEAN_BITS = {"uniform": 14 / 3, "mix": 0.8 + 0.6 * 4 + 0.3 * 2, "all2": 2, "all8": 8, "adaptive": 1.2 + 1.8 + 0.8}


def work(case):
    kind, dim, send = case["kind"], case["dim"], case["send"]
    if kind == "reassign":
        # a beta and a peer in, a width out; the plan's device arrays; a sort's comparisons
        return {"bytes": send * (4 + 4 + 1 + 4 + 1 + 8 + 4 + 4), "flops": 10 * send}
    row, packed = 4 * dim, dim * _MEAN_BITS[case["bits"]] / 8
    if kind == "gradients":
        # messages and their index entries in; the rows they fall on in and out
        hit = case["rows"] * (1 - math.exp(-send / case["rows"]))
        return {"bytes": send * (packed + 8 + 17) + hit * 2 * row, "flops": 3 * send * dim}
    sent = send * (row + packed + 8 + 13 + 8)           # row, index entries and alpha in; codes, (Z, S) and beta out
    received = send * (packed + 8 + 17 + row)
    flops = send * dim * (6 + 2)                        # min, max, subtract, multiply, round, pack; multiply, add
    if kind == "messages":
        return {"bytes": sent + received, "flops": flops}
    rows_in, rows_out = case["rows"] + case["halo"], case["rows"]
    if kind == "step" and case["backward"]:
        rows_in, rows_out = rows_out, rows_in
        received = send * (packed + 8 + 17) + case["rows"] * (1 - math.exp(-send / case["rows"])) * 2 * row \
            if case["receive"] else 0
    if kind == "step":
        received += 2 * send * (packed + 8)             # the exchange (here: a copy)
        if case["fused"]:
            received -= send * row
    return {"bytes": sent + received + case["edges"] * 8 + rows_in * row + rows_out * (row + 8),
            "flops": flops + 2 * case["edges"] * dim}


def tolerance(case):
    if case["kind"] in ("messages", "gradients", "reassign"):
        return "exact"
    if case["kind"] == "step" and case["backward"]:
        # what is quantised are sums: where one of them moves by its rounding error, a code next to a threshold moves by
        # one (8 bits: 255 steps times about 3e-7 of the codes); with the received messages added, such a step of
        # 1/255 of a row's range shows in the output
        return {"rel": 5e-4, "max": 0.4, "differ": 1e-3} if case["receive"] else {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
