"""The work a user of this package has it do, as cases that can be timed.

A case is a dict of plain values.  ``kind`` says which public entry points a pass goes through:

* ``layer``     heteroconv_fwd, then heteroconv_bwd, of one HeteroConv layer on one circuit graph
* ``ops``       the building blocks by themselves: dr_topk x2, dr_spmm_fwd x3, dr_spmm_bwd x3 (or the planned form)
* ``train``     hgnn_train_step over a batch of sub-graphs, stacked (hgnn_create_batched) or streamed (hgnn_create)
* ``setup``     what every new graph needs on the device: dr_csr_normalize and dr_csr_transpose of the three relations
* ``pipeline``  sub-graphs in host memory through dr_pipeline slots, a layer forward and backward on each

Graphs are drawn on the GPU from the same laws as ``circuit_synth/generate.py``: cells on a grid, ``near`` sources
distinct cells of a window around the destination, nets of 2 + Geometric members drawn uniformly from the cells, a
small share of high-fanout nets, ``pinned`` the transpose pattern of ``pins``.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2508_16769_amd as P

# ----------------------------------------------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------------------------------------------

# in-degree laws of `near`: (mean, draw); the power law is the one of the 1.2 M-cell design (4 .. 256, alpha = 2.2)
POWER_ALPHA, POWER_MIN, POWER_MAX = 2.2, 4, 256
NET_MEAN = {"low": 3.0, "high": 3.5}      # mean of the geometric part of a net's degree


def listed():
    return [
        # one layer on a toy or a freshly cut corner of a design: launches and latency are all there is
        dict(name="layer_tiny", kind="layer", cells=2048, nets=1024, near="const8", net="low", evil=0.0, D=64, k=16, placed=True),
        # one layer on a small block, hidden width 64
        dict(name="layer_small", kind="layer", cells=60_000, nets=40_000, near="poisson10", net="low", evil=0.0, D=64, k=16,
             placed=True),
        # one layer on a mid-size design with a few clock- and reset-like nets, hidden width 128
        dict(name="layer_medium", kind="layer", cells=250_000, nets=180_000, near="poisson12", net="high", evil=0.001, D=128, k=32,
             placed=True),
        # one layer on a whole full-chip graph
        dict(name="layer_large", kind="layer", cells=1_200_000, nets=900_000, near="powerlaw", net="high", evil=0.002, D=128, k=32,
             placed=True),
        # sizes that fit no tile, width 96, one K per edge type as the K profiling picks them, no placement at hand
        dict(name="layer_per_relation", kind="layer", cells=33_331, nets=24_989, near="poisson10", net="low", evil=0.0, D=96, k=16,
             k_pins=24, k_pinned=8, placed=False),
        # a training step of a 3-layer model over a batch of eight sampled sub-graphs, stacked into one
        dict(name="train_batched", kind="train", graphs=8, cells=20_000, nets=14_000, near="poisson10", net="low", evil=0.0, D=128,
             k=32, layers=3, batched=True),
        # the same for sub-graphs of unequal sizes on one stream each, two layers
        dict(name="train_streamed", kind="train", graphs=4, cells=13_337, nets=9_001, near="poisson10", net="low", evil=0.0, D=64,
             k=16, layers=2, batched=False),
        # the message-passing kernels alone on the full-chip graph (the benchmark's timed region), near^T on staged tiles
        dict(name="ops_large_k32", kind="ops", cells=1_200_000, nets=900_000, near="powerlaw", net="high", evil=0.002, D=128, k=32,
             placed=True),
        # the smallest width of the k sweep, mid-size design
        dict(name="ops_medium_k8", kind="ops", cells=250_000, nets=180_000, near="poisson12", net="high", evil=0.001, D=128, k=8,
             placed=True),
        # widths that fill no vector: D = 100, k = 25
        dict(name="ops_ragged", kind="ops", cells=45_677, nets=31_991, near="poisson10", net="low", evil=0.0, D=100, k=25,
             placed=False),
        # edge values and transposes of a mid-size design that has just been read
        dict(name="setup_medium", kind="setup", cells=250_000, nets=180_000, near="poisson12", net="high", evil=0.001),
        # training sub-graphs streamed from host memory through two pipeline slots
        dict(name="pipeline", kind="pipeline", graphs=4, cells=20_000, nets=14_000, near="poisson10", net="low", evil=0.0, D=128,
             k=32, slots=2, threads=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "ops", "ops", "ops", "train", "setup", "pipeline"])
    graph = dict(near=rng.choice(["const8", "poisson10", "poisson12", "powerlaw"]), net=rng.choice(["low", "high"]))
    if kind in ("train", "pipeline"):
        cells = _log_int(rng, 3_000, 20_000)
        # sampled sub-graphs: no high-fanout nets, moderate degrees
        graph["near"] = rng.choice(["const8", "poisson10", "poisson12"])
        case = dict(kind=kind, graphs=rng.randint(2, 8), cells=cells, nets=max(1, int(cells * rng.uniform(0.5, 0.8))), evil=0.0,
                    **graph)
        case["D"] = rng.choice([64, 96, 128])
        case["k"] = rng.choice([8, 16, 32])
        if kind == "train":
            case.update(layers=rng.choice([2, 3]), batched=rng.random() < 0.5)
        else:
            case.update(graphs=rng.randint(2, 4), slots=rng.choice([2, 3]), threads=2)
        return case
    cells = _log_int(rng, 2_000, 1_100_000)
    case = dict(kind=kind, cells=cells, nets=max(1, int(cells * rng.uniform(0.5, 0.75))),
                evil=rng.choice([0.0, 0.001, 0.002]) if cells >= 50_000 else 0.0, **graph)
    if kind == "setup":
        return case
    if kind == "layer":
        case["D"] = rng.choice([32, 64, 96, 128, 128])
        widths = [w for w in (4, 8, 12, 16, 24, 32) if w <= case["D"] // 2]
        case["k"] = rng.choice(widths)
        if rng.random() < 0.25:
            case["k_pins"], case["k_pinned"] = rng.choice(widths), rng.choice(widths)
        case["placed"] = rng.random() < 0.7
    else:
        case["D"] = rng.choice([32, 64, 96, 100, 128, 128])
        widths = [w for w in (5, 8, 16, 20, 25, 32, 64) if w <= case["D"] // 2]
        case["k"] = rng.choice(widths)
        case["placed"] = case["D"] % 32 == 0 and rng.random() < 0.7
    return case


# ----------------------------------------------------------------------------------------------------------------
# graphs, on the GPU
# ----------------------------------------------------------------------------------------------------------------

class _Pattern:
    def __init__(self, n_rows, n_cols, rowptr, colidx):
        self.n_rows, self.n_cols, self.rowptr, self.colidx = n_rows, n_cols, rowptr, colidx


def _grid(cells):
    width = max(1, int(math.ceil(math.sqrt(1.2 * cells))))
    return width, -(-cells // width)


def _csr(rows, cols, n_rows, n_cols):
    rowptr = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(rows, minlength=n_rows), 0, out=rowptr[1:])
    return _Pattern(n_rows, n_cols, rowptr.to(torch.int32), cols.to(torch.int32))


def _near_degrees(law, n, gen):
    if law == "const8":
        return torch.full((n,), 8, dtype=torch.int64, device="cuda")
    if law.startswith("poisson"):
        lam = torch.full((n,), float(law[len("poisson"):]), device="cuda")
        return torch.poisson(lam, generator=gen).to(torch.int64)
    support = torch.arange(POWER_MIN, POWER_MAX + 1, dtype=torch.float64, device="cuda")
    pmf = support ** (-POWER_ALPHA)
    cdf = torch.cumsum(pmf / pmf.sum(), 0)
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    return torch.clamp(torch.searchsorted(cdf, u, right=True), max=support.numel() - 1) + POWER_MIN


def _to_total(deg, total, least, gen):
    """Degrees changed by one here and there until they add up to the expected number of edges."""
    while (off := total - int(deg.sum())) != 0:
        rows = torch.nonzero(deg > least).flatten() if off < 0 else torch.arange(deg.numel(), device="cuda")
        who = rows[torch.randperm(rows.numel(), device="cuda", generator=gen)[:abs(off)]]
        deg[who] += 1 if off > 0 else -1
    return deg


def _make_near(cells, law, edges, gen):
    """Every destination cell takes `degree` distinct sources from the (2r+1)^2 window around it."""
    width, height = _grid(cells)
    deg = _to_total(_near_degrees(law, cells, gen), edges, 1, gen)
    radius = torch.clamp(torch.ceil(torch.sqrt(deg.to(torch.float64) + 1.0)).to(torch.int64) - 1, min=2)
    # a window that reaches the grid's last, partly filled row is made one wider, so that it has enough candidates
    radius = radius + (torch.arange(cells, device="cuda") // width + radius >= height - 1).to(torch.int64)
    keys = []
    for r in torch.unique(radius).tolist():
        ids = torch.nonzero((radius == r) & (deg > 0)).flatten()
        side = 2 * r + 1
        off = torch.arange(side * side, device="cuda")
        dx, dy = off % side - r, off // side - r
        chunk = max(1, (64 << 20) // (side * side))
        for s in range(0, ids.numel(), chunk):
            cid = ids[s:s + chunk]
            nx, ny = (cid % width)[:, None] + dx, (cid // width)[:, None] + dy
            nid = ny * width + nx
            out = (nx < 0) | (nx >= width) | (ny < 0) | (ny >= height) | (nid >= cells) | (nid == cid[:, None])
            score = torch.rand(nid.shape, device="cuda", generator=gen).masked_fill_(out, 2.0)
            d = deg[cid]
            score, order = torch.sort(score, dim=1)
            take = (torch.arange(side * side, device="cuda") < d[:, None]) & (score < 2.0)
            keys.append((cid[:, None] * cells + torch.gather(nid, 1, order))[take])
    key = torch.sort(torch.cat(keys))[0]
    return _csr(key // cells, key % cells, cells, cells)


def _make_pins(nets, cells, mean, evil, edges, gen):
    """Rows are nets, columns their member cells (distinct, uniform)."""
    u = torch.rand(nets, dtype=torch.float64, device="cuda", generator=gen)
    deg = 2 + torch.clamp(torch.ceil(torch.log1p(-u) / math.log1p(-1.0 / mean)), min=1).to(torch.int64)
    if evil == 0.0:
        deg = torch.clamp(deg, max=64)
    n_evil = int(round(evil * nets))
    if n_evil:
        who = torch.randperm(nets, device="cuda", generator=gen)[:n_evil]
        deg[who] = torch.randint(200, 2001, (n_evil,), device="cuda", generator=gen)
    deg = _to_total(deg, edges, 2, gen)
    rows = torch.repeat_interleave(torch.arange(nets, device="cuda"), deg)
    key = rows * cells + torch.randint(0, cells, (rows.numel(),), device="cuda", generator=gen)
    while True:                                          # members drawn twice are drawn again
        key = torch.sort(key)[0]
        twice = torch.nonzero(key[1:] == key[:-1]).flatten() + 1
        if twice.numel() == 0:
            break
        key[twice] = key[twice] // cells * cells + torch.randint(0, cells, (twice.numel(),), device="cuda", generator=gen)
    return _csr(key // cells, key % cells, nets, cells)


def _cell_order(cells):
    """The cells along the Z-order curve of their grid coordinates."""
    width, _ = _grid(cells)
    ids = torch.arange(cells, device="cuda")

    def spread(v):
        for shift, mask in ((8, 0x00FF00FF), (4, 0x0F0F0F0F), (2, 0x33333333), (1, 0x55555555)):
            v = (v | (v << shift)) & mask
        return v

    return torch.argsort(spread(ids % width) | (spread(ids // width) << 1), stable=True).to(torch.int32)


def _normalize(mode, pat, ws=None, vals=None):
    vals = torch.empty(pat.colidx.numel(), dtype=torch.float32, device="cuda") if vals is None else vals
    P.dr_csr_normalize(mode, pat.n_rows, pat.n_cols, pat.rowptr, pat.colidx, vals, ws)
    return vals


def _workspace(nbytes):
    return torch.empty(max(256, nbytes), dtype=torch.uint8, device="cuda")


def _patterns(case, gen):
    near_edges, pins_edges = _edges(case, case["cells"], case["nets"])
    near = _make_near(case["cells"], case["near"], near_edges, gen)
    pins = _make_pins(case["nets"], case["cells"], NET_MEAN[case["net"]], case["evil"], pins_edges, gen)
    return near, pins


def _relations(near, pins):
    """The three relations with their edge values."""
    t = P.device_transpose(P.Csr(pins.n_rows, pins.n_cols, pins.rowptr, pins.colidx, None))
    pinned = _Pattern(t.n_rows, t.n_cols, t.rowptr, t.colidx)
    out = []
    for pat, mode in ((near, P.DR_NORM_MEAN), (pins, P.DR_NORM_MEAN), (pinned, P.DR_NORM_SYM)):
        ws = _workspace(P.dr_csr_normalize_workspace_bytes(mode, pat.n_rows, pat.n_cols, pat.colidx.numel()))
        out.append(P.Csr(pat.n_rows, pat.n_cols, pat.rowptr, pat.colidx, _normalize(mode, pat, ws)))
    return out


def _normal(shape, gen):
    return torch.randn(shape, device="cuda", generator=gen)


def _weights(D, gen):
    bound = math.sqrt(6.0 / (D + D))
    return {n: torch.empty((D, D), device="cuda").uniform_(-bound, bound, generator=gen) for n in P.WEIGHT_NAMES}


def _layer_io(Nc, Nn, D, gen):
    """Outputs and upstream gradients of one layer pass, and the merge mask its backward reads."""
    return dict(
        Y_cell=torch.empty((Nc, D), device="cuda"), Y_net=torch.empty((Nn, D), device="cuda"),
        dY_cell=_normal((Nc, D), gen), dY_net=_normal((Nn, D), gen),
        dX_cell=torch.empty((Nc, D), device="cuda"), dX_net=torch.empty((Nn, D), device="cuda"),
        dW={n: torch.empty((D, D), device="cuda") for n in P.WEIGHT_NAMES},
        # The forward writes saved["mask"]; the backward is given this one, as likely to name either branch.  Which branch
        # wins where both agree to the last bits is decided by rounding, and one element of the gradient is then another
        # number altogether: with a mask of the case's own, a pass's gradients are a matter of arithmetic alone.
        mask=torch.randint(0, 2, (Nc, D), dtype=torch.uint8, device="cuda", generator=gen))


# ----------------------------------------------------------------------------------------------------------------
# prepare and run
# ----------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return _PREPARE[case["kind"]](case, gen)


def run(state):
    return _RUN[state["kind"]](state)


def _prepare_layer(case, gen):
    D = case["D"]
    near, pins = _patterns(case, gen)
    rel = _relations(near, pins)
    if "k_pins" in case:
        layer = P.HeteroConv(*rel, D, per_relation=(case["k"], case["k_pins"], case["k_pinned"]))
    else:
        layer = P.HeteroConv(*rel, D, case["k"], case["k"])
    if case["placed"]:
        layer.heteroconv_set_cell_order(_cell_order(case["cells"]))
    st = dict(kind="layer", layer=layer, X_cell=_normal((layer.Nc, D), gen), X_net=_normal((layer.Nn, D), gen), W=_weights(D, gen),
              saved=layer.alloc_saved(), **_layer_io(layer.Nc, layer.Nn, D, gen))
    st["saved_bwd"] = dict(st["saved"], mask=st.pop("mask"))
    return st


def _run_layer(st):
    layer = st["layer"]
    layer.heteroconv_fwd(st["X_cell"], st["X_net"], st["W"], st["Y_cell"], st["Y_net"], st["saved"])
    layer.heteroconv_bwd(st["dY_cell"], st["dY_net"], st["W"], st["saved_bwd"], st["dX_cell"], st["dX_net"], st["dW"])
    return dict(Y_cell=st["Y_cell"], Y_net=st["Y_net"], saved=st["saved"], dX_cell=st["dX_cell"], dX_net=st["dX_net"], dW=st["dW"])


def _prepare_ops(case, gen):
    D, k, n = case["D"], case["k"], dict(cell=case["cells"], net=case["nets"])
    rel = _relations(*_patterns(case, gen))
    rel_t = [P.device_transpose(A) for A in rel]
    dst, src = ("cell", "net", "cell"), ("cell", "cell", "net")
    st = dict(kind="ops", D=D, k=k, rel=rel, rel_t=rel_t, src=src, dst=dst,
              X={t: _normal((n[t], D), gen) for t in n}, dH=[_normal((n[t], D), gen) for t in dst],
              vals={t: torch.empty((n[t], k), device="cuda") for t in n},
              idx={t: torch.empty((n[t], k), dtype=torch.int16, device="cuda") for t in n},
              H=[torch.empty((n[t], D), device="cuda") for t in dst], G=[torch.empty((n[t], k), device="cuda") for t in src])
    st["plan"] = P.SpmmPlan(rel_t[0], D, _cell_order(case["cells"])) if case["placed"] else None
    return st


def _run_ops(st):
    D, k = st["D"], st["k"]
    for t in ("cell", "net"):
        P.dr_topk(st["X"][t], k, st["vals"][t], st["idx"][t])
    for A, src, H in zip(st["rel"], st["src"], st["H"]):
        P.dr_spmm_fwd(A, st["vals"][src], st["idx"][src], D, k, H)
    for r, (At, src, dH, G) in enumerate(zip(st["rel_t"], st["src"], st["dH"], st["G"])):
        if r == 0 and st["plan"] is not None:
            st["plan"].dr_spmm_bwd_planned(dH, st["idx"][src], k, G)
        else:
            P.dr_spmm_bwd(At, dH, st["idx"][src], D, k, G)
    return dict(vals=st["vals"], idx=st["idx"], H=st["H"], G=st["G"])


def _sizes(case, q):
    """Sub-graph q of a batch: streamed batches hold sub-graphs of unequal sizes, stacked ones of equal size."""
    if case.get("batched", False):
        return case["cells"], case["nets"]
    scale = 1.0 - 0.07 * (q % 4)
    return max(600, int(case["cells"] * scale)), max(300, int(case["nets"] * scale))


def _prepare_train(case, gen):
    D, graphs, keep = case["D"], [], []
    for q in range(case["graphs"]):
        cells, nets = _sizes(case, q)
        rel = _relations(*_patterns(dict(case, cells=cells, nets=nets), gen))
        graphs.append(P.HeteroConv(*rel, D, case["k"], case["k"]))
    model = P.Hgnn(graphs, case["layers"], batched=case["batched"])
    nc, nn = sum(g.Nc for g in graphs), sum(g.Nn for g in graphs)
    xc, xn, tg = _normal((nc, D), gen), _normal((nn, D), gen), _normal((nc,), gen)
    keep += [xc, xn, tg]
    split = lambda t, sizes: list(torch.split(t, sizes))          # noqa: E731  one batch tensor, a view per sub-graph
    n_par = P.hgnn_num_params(case["layers"], D)
    bound = math.sqrt(6.0 / (D + D))
    theta = torch.empty(n_par, device="cuda").uniform_(-bound, bound, generator=gen)
    return dict(kind="train", model=model, keep=keep, X_cell=split(xc, [g.Nc for g in graphs]), X_net=split(xn, [g.Nn for g in graphs]),
                target=split(tg, [g.Nc for g in graphs]), theta=theta, m=torch.zeros_like(theta), v=torch.zeros_like(theta),
                grad=torch.empty_like(theta), loss=torch.empty(1, device="cuda"), step=0)


def _run_train(st):
    st["step"] += 1
    st["model"].hgnn_train_step(st["X_cell"], st["X_net"], st["target"], st["theta"], st["m"], st["v"], 2e-4, 0.9, 0.999, 1e-8, 1e-5,
                                st["step"], st["grad"], st["loss"])
    return dict(loss=st["loss"], grad=st["grad"], theta=st["theta"], m=st["m"], v=st["v"])


def _prepare_setup(case, gen):
    near, pins = _patterns(case, gen)
    t = P.device_transpose(P.Csr(pins.n_rows, pins.n_cols, pins.rowptr, pins.colidx, None))
    pinned = _Pattern(t.n_rows, t.n_cols, t.rowptr, t.colidx)
    st = dict(kind="setup", rel=[])
    for pat, mode in ((near, P.DR_NORM_MEAN), (pins, P.DR_NORM_MEAN), (pinned, P.DR_NORM_SYM)):
        E = pat.colidx.numel()
        A = P.Csr(pat.n_rows, pat.n_cols, pat.rowptr, pat.colidx, torch.empty(E, device="cuda"))
        st["rel"].append(dict(
            A=A, mode=mode, ws_n=_workspace(P.dr_csr_normalize_workspace_bytes(mode, pat.n_rows, pat.n_cols, E)),
            ws_t=_workspace(P.dr_csr_transpose_workspace_bytes(pat.n_rows, pat.n_cols, E)),
            t_rowptr=torch.empty(pat.n_cols + 1, dtype=torch.int32, device="cuda"),
            t_colidx=torch.empty(E, dtype=torch.int32, device="cuda"), t_vals=torch.empty(E, device="cuda")))
    return st


def _run_setup(st):
    out = []
    for r in st["rel"]:
        A = r["A"]
        P.dr_csr_normalize(r["mode"], A.n_rows, A.n_cols, A.rowptr, A.colidx, A.vals, r["ws_n"])
        P.dr_csr_transpose(A, r["t_rowptr"], r["t_colidx"], r["t_vals"], r["ws_t"])
        out.append((A.vals, r["t_rowptr"], r["t_colidx"], r["t_vals"]))
    return out


def _prepare_pipeline(case, gen):
    D, k = case["D"], case["k"]
    host, io = [], []
    for q in range(case["graphs"]):
        cells, nets = _sizes(case, q)
        near, pins = _patterns(dict(case, cells=cells, nets=nets), gen)
        xc, xn = _normal((cells, D), gen), _normal((nets, D), gen)
        host.append([t.cpu().numpy() for t in (near.rowptr, near.colidx, pins.rowptr, pins.colidx, xc, xn)])
        io.append(_layer_io(cells, nets, D, gen))
    most = [max(int(g[i].shape[0]) for g in host) for i in range(4)]
    Nc, Nn = most[0] - 1, most[2] - 1
    pipe = P.Pipeline(case["slots"], case["threads"], Nc, Nn, most[1], most[3], D, k, k)
    saved = dict(vals_cell=torch.empty((Nc, k), device="cuda"), idx_cell=torch.empty((Nc, k), dtype=torch.int16, device="cuda"),
                 vals_net=torch.empty((Nn, k), device="cuda"), idx_net=torch.empty((Nn, k), dtype=torch.int16, device="cuda"),
                 H_near=torch.empty((Nc, D), device="cuda"), H_pins=torch.empty((Nn, D), device="cuda"),
                 H_pinned=torch.empty((Nc, D), device="cuda"), mask=torch.empty((Nc, D), dtype=torch.uint8, device="cuda"))
    return dict(kind="pipeline", pipe=pipe, slots=case["slots"], host=host, io=io, W=_weights(D, gen), saved=saved)


def _run_pipeline(st):
    pipe, slots, host, saved = st["pipe"], st["slots"], st["host"], st["saved"]
    for q in range(min(slots, len(host))):
        pipe.dr_pipeline_submit(q, *host[q])
    out = []
    for q, io in enumerate(st["io"]):
        layer, xc, xn = pipe.dr_pipeline_acquire(q % slots)
        layer.heteroconv_fwd(xc, xn, st["W"], io["Y_cell"], io["Y_net"], saved)
        layer.heteroconv_bwd(io["dY_cell"], io["dY_net"], st["W"], dict(saved, mask=io["mask"]), io["dX_cell"], io["dX_net"], io["dW"])
        pipe.dr_pipeline_release(q % slots)
        if q + slots < len(host):
            pipe.dr_pipeline_submit((q + slots) % slots, *host[q + slots])
        out.append((io["Y_cell"], io["Y_net"], io["dX_cell"], io["dX_net"], io["dW"]))
    return out


_PREPARE = dict(layer=_prepare_layer, ops=_prepare_ops, train=_prepare_train, setup=_prepare_setup, pipeline=_prepare_pipeline)
_RUN = dict(layer=_run_layer, ops=_run_ops, train=_run_train, setup=_run_setup, pipeline=_run_pipeline)


# ----------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------------------------

def _edges(case, cells, nets):
    """Number of edges of (near, pins): what the degree laws expect."""
    law = case["near"]
    if law == "powerlaw":
        d = np.arange(POWER_MIN, POWER_MAX + 1, dtype=np.float64)
        p = d ** (-POWER_ALPHA)
        mean = float((d * p).sum() / p.sum())
    else:
        mean = float(law[len("const"):] if law.startswith("const") else law[len("poisson"):])
    net = (1.0 - case["evil"]) * (2.0 + NET_MEAN[case["net"]]) + case["evil"] * min(1100.0, float(cells))
    return int(round(mean * cells)), int(round(net * nets))


def _csr_bytes(rows, edges):
    return 4 * (rows + 1) + 8 * edges


def _layer_work(case, cells, nets):
    """One layer forward and backward: inputs, relations and their transposes, what is saved, outputs and gradients, once."""
    D, k = case["D"], case["k"]
    k_pins, k_pinned = case.get("k_pins", k), case.get("k_pinned", k)
    near, pins = _edges(case, cells, nets)
    sel_c = k + (k_pins if k_pins != k else 0)
    sel_n = k_pinned + (k_pins if "k_pins" in case and k_pins != k_pinned else 0)
    graph = 2 * _csr_bytes(cells, near) + _csr_bytes(nets, pins) + 2 * _csr_bytes(cells, pins) + _csr_bytes(nets, pins)
    fwd = 4 * D * (cells + nets) + 6 * (cells * sel_c + nets * sel_n) + 4 * D * (2 * cells + nets) + cells * D + 4 * D * (cells + nets)
    bwd = 4 * D * (cells + nets) + cells * D + 4 * D * (cells + nets)
    weights = 4 * 15 * D * D
    dense = 2.0 * D * D * (2 * cells + 2 * nets + cells) * 3
    sparse = 4.0 * (near * k + pins * k_pins + pins * k_pinned)
    return graph + fwd + bwd + weights, dense + sparse, (graph, weights)


def work(case):
    kind, cells, nets = case["kind"], case["cells"], case["nets"]
    if kind == "layer":
        b, f, _ = _layer_work(case, cells, nets)
        return {"bytes": b, "flops": f}
    if kind == "ops":
        D, k = case["D"], case["k"]
        near, pins = _edges(case, cells, nets)
        b = 4 * D * (cells + nets) + 6 * k * (cells + nets)                                             # D-ReLU
        b += _csr_bytes(cells, near) + _csr_bytes(nets, pins) + _csr_bytes(cells, pins) + 4 * D * (2 * cells + nets)      # forward
        b += _csr_bytes(cells, near) + _csr_bytes(cells, pins) + _csr_bytes(nets, pins) + 4 * D * (2 * cells + nets)      # backward
        b += 4 * k * (2 * cells + nets)
        return {"bytes": b, "flops": 4.0 * k * (near + 2 * pins)}
    if kind == "setup":
        near, pins = _edges(case, cells, nets)
        rows = cells + nets + cells
        return {"bytes": 4 * rows + 4 * (near + 2 * pins) + 4 * (near + 2 * pins) + 4 * (cells + cells + nets) + 8 * (near + 2 * pins),
                "flops": 0.0}
    b = f = 0.0
    for q in range(case["graphs"]):
        c, n = _sizes(case, q)
        lb, lf, (graph, weights) = _layer_work(case, c, n)
        if kind == "pipeline":
            near, pins = _edges(case, c, n)
            b += lb + _csr_bytes(c, near) - 4 * near + _csr_bytes(n, pins) - 4 * pins
            f += lf
        else:
            # the relations are read by every layer; nobody reads the first layer's dX or the last layer's net output
            D = case["D"]
            b += case["layers"] * (lb - weights) - 4 * D * (c + n) - 4 * D * (3 * n)
            f += case["layers"] * lf - 2.0 * D * D * (3 * c + 2 * n) - 4.0 * D * D * n * 3
    if kind == "train":
        b += 4 * 8 * case["layers"] * 5 * case["D"] ** 2
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "setup":
        return "exact"
    if case["kind"] == "train":
        # 32-bit sums, but a rounding of the first layer decides, at about one element in ten million, which branch of the
        # merge wins or which entry D-ReLU of the next layer keeps: a share f of the terms of a gradient is then another
        # number, which moves it by about sqrt(f)
        return {"rel": 3e-3, "max": 0.1}
    # 32-bit sums of up to a few thousand terms; the merge mask names the larger of two sums
    return {"rel": 1e-5, "max": 4e-4, "differ": 1e-5}
