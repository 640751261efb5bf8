"""Input gradients of hub cells: rows whose records come from two transposed relations with the cell's own piece between them
(near, self term, pins) and are long enough to be walked by a wavefront (more than 32) or by a whole workgroup (more than
256).  The lengths put the ends of the lists on and next to the places where a row is cut: the 32 and 256 of the dispatch, the
quarters of a workgroup's row and its chunks of 256 records.  Without a cell order, with one width and with widths of their
own, as a layer and behind a ReLU (the gate on the gradient) as the upper layer of a model."""
import numpy as np
import pytest
import torch

import paper_2508_16769_amd as P
from gpu_util import dev, host_idx, say

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 31, 32, 33, 127, 128, 255, 256, 257, 700, 1500]


def _relations(rng, Nc, Nn):
    """near (Nc x Nc), pins (Nn x Nc), pinned (Nc x Nn) as (rows, cols, values); hub cell h of the first len^2 cells is the
    source of LENGTHS[h // n] near and LENGTHS[h % n] pins entries, further cells of a few."""
    n = len(LENGTHS)
    out = np.concatenate([np.repeat(LENGTHS, n), rng.integers(0, 6, Nc - n * n)])       # near entries per source cell
    pin = np.concatenate([np.tile(LENGTHS, n), rng.integers(0, 4, Nc - n * n)])
    rel = []
    for src, rows in ((np.repeat(np.arange(Nc), out), Nc), (np.repeat(np.arange(Nc), pin), Nn)):
        dst = rng.integers(0, rows, len(src))
        order = np.lexsort((src, dst))
        rel.append((dst[order], src[order]))
    rel.append(tuple(a[np.lexsort((rel[1][0], rel[1][1]))] for a in (rel[1][1], rel[1][0])))
    return [(r, c, rng.uniform(0.05, 1.0, len(r)).astype(np.float32)) for r, c in rel]


def _csr(r, c, v, M, N):
    rp = np.zeros(M + 1, np.int32)
    np.cumsum(np.bincount(r, minlength=M), out=rp[1:])
    return P.Csr(M, N, dev(rp), dev(c.astype(np.int32)), dev(v))


def _scatter(r, c, v, dH, N):
    """A^T dH and the sum of the absolute values of its terms, fp64."""
    want, l1 = np.zeros((N, dH.shape[1])), np.zeros((N, dH.shape[1]))
    np.add.at(want, c, v[:, None].astype(np.float64) * dH[r])
    np.add.at(l1, c, v[:, None].astype(np.float64) * np.abs(dH[r]))
    return want, l1


def _expected(rel, dYc, dYn, mask, W, sel, gate, Nc, Nn):
    """dX of the cells and nets and the L1 norms of their terms.  dH rows are sums of 2 D products, formed before they are summed."""
    dZn, dZq = np.where(mask == 1, dYc, 0.0), np.where(mask == 0, dYc, 0.0)
    W = {n: w.astype(np.float64) for n, w in W.items()}
    on = {u: np.zeros((Nc if u in ("near", "pins") else Nn, dYc.shape[1])) for u in sel}
    for u, i in sel.items():
        np.put_along_axis(on[u], i.astype(np.int64), 1.0 if gate is None else (gate[u] > 0).astype(np.float64), axis=1)
    res = []
    for ab in (False, True):
        f = np.abs if ab else (lambda x: x)
        w = {n: f(x) for n, x in W.items()}
        k = 1 if ab else 0
        c = on["near"] * (f(dZn) @ w["self_near"].T + _scatter(*rel[0], f(dZn) @ w["neigh_near"].T, Nc)[k])
        c += on["pins"] * _scatter(*rel[1], f(dYn) @ w["neigh_pins"].T, Nc)[k]
        n = on["self"] * (f(dYn) @ w["self_pins"].T) + on["pinned"] * _scatter(*rel[2], f(dZq) @ w["pinned"].T, Nn)[k]
        res.append((c, n))
    return res


def _check(got, want, l1, what):
    # up to 3001 terms added in at least 8 partial sums of at most 376, each term a sum of 2 D <= 256 products (2^-23 of its L1
    # norm): (376 + 256) * 2^-24 = 3.8e-5; measured below 2e-6
    assert np.all(np.abs(got - want) <= 1e-5 * l1), (what, float((np.abs(got - want) / np.maximum(l1, 1e-300)).max()))


@pytest.mark.parametrize("mode", [P.DR_OVERLAP_ON, P.DR_OVERLAP_OFF])
@pytest.mark.parametrize("D,ks", [(32, (8, 8, 8)), (64, (16, 16, 16)), (128, (32, 32, 32)), (64, (16, 24, 8)), (128, (64, 64, 20)), (96, (70, 33, 70))])
def test_hub_cells_in_a_layer(D, ks, mode):
    Nc, Nn = 400, 300
    say(f"hubs D={D} k={ks} mode={mode}")
    rng = np.random.default_rng(D + sum(ks))
    f = lambda *s: rng.standard_normal(s).astype(np.float32)             # noqa: E731
    rel = _relations(rng, Nc, Nn)
    layer = P.HeteroConv(*(_csr(*r, m, n) for r, m, n in zip(rel, (Nc, Nn, Nc), (Nc, Nc, Nn))), D, per_relation=ks)
    layer.heteroconv_set_overlap(mode)
    W = {n: (f(D, D) / np.sqrt(D)).astype(np.float32) for n in P.WEIGHT_NAMES}
    Wd = {n: dev(w) for n, w in W.items()}
    saved = layer.alloc_saved()
    e = lambda *s: torch.full(s, float("nan"), device="cuda")            # noqa: E731
    dYc, dYn = f(Nc, D), f(Nn, D)
    layer.heteroconv_fwd(dev(f(Nc, D)), dev(f(Nn, D)), Wd, e(Nc, D), e(Nn, D), saved)
    dXc, dXn = e(Nc, D), e(Nn, D)
    layer.heteroconv_bwd(dev(dYc), dev(dYn), Wd, saved, dXc, dXn, {n: e(D, D) for n in P.WEIGHT_NAMES})
    torch.cuda.synchronize()
    sel = dict(near=host_idx(saved["idx_cell"]), pinned=host_idx(saved["idx_net"]))
    sel["pins"] = host_idx(saved["idx_cell_pins"]) if ks[1] != ks[0] else sel["near"]
    sel["self"] = host_idx(saved["idx_net_self"]) if ks[1] != ks[2] else sel["pinned"]
    (wc, wn), (lc, ln) = _expected(rel, dYc.astype(np.float64), dYn.astype(np.float64), saved["mask"].cpu().numpy(), W, sel, None, Nc, Nn)
    _check(dXc.cpu().numpy(), wc, lc, "dX_cell")
    _check(dXn.cpu().numpy(), wn, ln, "dX_net")
    layer.heteroconv_destroy()


@pytest.mark.parametrize("ks", [(60, 60, 60), (50, 64, 55), (70, 55, 70)])
def test_hub_cells_behind_a_relu(ks):
    """The upper layers of a model: dX is gated where the layer's input was not positive."""
    Nc, Nn, D = 400, 300, 96
    say(f"hubs behind a ReLU k={ks}")
    rng = np.random.default_rng(sum(ks))
    f = lambda *s: rng.standard_normal(s).astype(np.float32)             # noqa: E731
    rel = _relations(rng, Nc, Nn)
    layer = P.HeteroConv(*(_csr(*r, m, n) for r, m, n in zip(rel, (Nc, Nn, Nc), (Nc, Nc, Nn))), D, per_relation=ks)
    L = 3
    model = P.Hgnn([layer], L, batched=False)
    theta0 = ((f(P.hgnn_num_params(L, D)) - 0.1) * 0.05).astype(np.float32)       # more outputs below zero than selected
    theta = dev(theta0)
    z = lambda: torch.zeros_like(theta)                                  # noqa: E731
    X, Xn, target, loss, grad, m, v = dev(f(Nc, D)), dev(f(Nn, D)), dev(f(Nc)), torch.zeros(1, device="cuda"), z(), z(), z()
    model.hgnn_train_step([X], [Xn], [target], theta, m, v, 1e-3, 0.9, 0.999, 1e-8, 0.0, 1, grad, loss)
    torch.cuda.synchronize()
    for l in (1, 2):
        b = model.hgnn_get_layer_buffers(0, l)
        W = {n: theta0[(5 * l + i) * D * D:(5 * l + i + 1) * D * D].reshape(D, D) for i, n in enumerate(P.WEIGHT_NAMES)}
        near, pins = ("cell", "cell_pins" if ks[1] != ks[0] else "cell")
        pinned, self_ = ("net", "net_self" if ks[1] != ks[2] else "net")
        uses = dict(near=near, pins=pins, self=self_, pinned=pinned)
        sel = {u: host_idx(b["idx_" + t]) for u, t in uses.items()}
        gate = {u: b["vals_" + t].cpu().numpy() for u, t in uses.items()}
        assert all((g <= 0).any() and (g > 0).any() for g in gate.values())
        dYc, dYn = b["dY_cell"].cpu().numpy().astype(np.float64), b["dY_net"].cpu().numpy().astype(np.float64)
        (wc, wn), (lc, ln) = _expected(rel, dYc, dYn, b["mask"].cpu().numpy(), W, sel, gate, Nc, Nn)
        _check(b["dX_cell"].cpu().numpy(), wc, lc, f"dX_cell of layer {l}")
        _check(b["dX_net"].cpu().numpy(), wn, ln, f"dX_net of layer {l}")
    model.hgnn_destroy()
    layer.heteroconv_destroy()
