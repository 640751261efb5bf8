"""The layer's dense products (three bf16 parts per fp32 operand) where their tiles and dispatch change: row counts around
the row tile of every width (128 rows at D = 32, 64 at D = 64, 32 at D = 96 and 128), selections wider than the pairs a
thread holds in registers, widths of their own per relation, and values at the ends of the fp32 range."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_16769_amd as P
from gpu_util import dev, random_csr, say

pytestmark = pytest.mark.gpu

WIDTHS = [(32, 4, 20, 32), (64, 16, 16, 16), (64, 40, 8, 64), (96, 33, 12, 33), (128, 32, 32, 32), (128, 70, 128, 16)]


def _run(Nc, Nn, D, ks, rng, X_cell, X_net, W, dY_cell, dY_net, edges=True, dup=False):
    """A layer pass; returns everything as fp64 numpy, with H and the selections the dense products read.  Without edges the
    products see the inputs alone."""
    deg = 3 if edges else 0
    near, pins, pinned = (random_csr(rng, m, n, deg, dup=dup) for m, n in ((Nc, Nc), (Nn, Nc), (Nc, Nn)))
    rel = [P.Csr(m, n, *(dev(a) for a in r)) for m, n, r in ((Nc, Nc, near), (Nn, Nc, pins), (Nc, Nn, pinned))]
    layer = P.HeteroConv(*rel, D, per_relation=ks)
    saved = layer.alloc_saved()
    Wd = {n: dev(W[n]) for n in P.WEIGHT_NAMES}
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")          # noqa: E731
    out = dict(Y_cell=nan(Nc, D), Y_net=nan(Nn, D), dX_cell=nan(Nc, D), dX_net=nan(Nn, D))
    dW = {n: nan(D, D) for n in P.WEIGHT_NAMES}
    layer.heteroconv_fwd(dev(X_cell), dev(X_net), Wd, out["Y_cell"], out["Y_net"], saved)
    layer.heteroconv_bwd(dev(dY_cell), dev(dY_net), Wd, saved, out["dX_cell"], out["dX_net"], dW)
    torch.cuda.synchronize()
    got = {n: t.cpu().numpy().astype(np.float64) for n, t in {**out, **dW, **{n: saved[n] for n in ("H_near", "H_pins", "H_pinned")}}.items()}
    got["mask"] = saved["mask"].cpu().numpy()
    k_near, k_pins, k_pinned = ks
    if not edges:
        layer.heteroconv_destroy()
        return got
    got["Xs_cell"] = oracle.densify(*oracle.topk(X_cell, k_near), D)
    got["Xs_self"] = oracle.densify(*oracle.topk(X_net, k_pins), D)
    got["sel"] = dict(near=oracle.topk(X_cell, k_near)[1], pins=oracle.topk(X_cell, k_pins)[1],
                      self=oracle.topk(X_net, k_pins)[1], pinned=oracle.topk(X_net, k_pinned)[1])
    layer.heteroconv_destroy()
    return got, near, pins, pinned


def _within(got, terms, what, n):
    """got against sum of A @ B over `terms`: n summed products, each off by at most 2^-24 of the running sum, plus the
    products a split leaves out (2^-24 of each): n * 2^-23 of the L1 norm of the terms bounds both, with 4 as the floor."""
    want = sum(a @ b for a, b in terms)
    l1 = sum(np.abs(a) @ np.abs(b) for a, b in terms)
    assert np.all(np.abs(got - want) <= max(n, 4) * 2.0 ** -23 * l1), (what, float((np.abs(got - want) / np.maximum(l1, 1e-300)).max()))


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 63, 65, 128, 129, 257])
@pytest.mark.parametrize("D,k_near,k_pins,k_pinned", WIDTHS)
def test_products_at_tile_edges(D, k_near, k_pins, k_pinned, rows):
    Nc, Nn = rows, max(1, rows - 1)
    say(f"dense rows={rows} D={D} k=({k_near},{k_pins},{k_pinned})")
    rng = np.random.default_rng(1000 * D + rows)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)             # noqa: E731
    W = {n: (f(D, D) / np.sqrt(D)).astype(np.float32) for n in P.WEIGHT_NAMES}
    dYc, dYn = f(Nc, D), f(Nn, D)
    got, near, pins, pinned = _run(Nc, Nn, D, (k_near, k_pins, k_pinned), rng, f(Nc, D), f(Nn, D), W, dYc, dYn)
    W = {n: w.astype(np.float64) for n, w in W.items()}
    dYc, dYn = dYc.astype(np.float64), dYn.astype(np.float64)
    # forward: the merge takes the larger branch, and the mask says which
    zn = [(got["Xs_cell"], W["self_near"]), (got["H_near"], W["neigh_near"])]
    zq = [(got["H_pinned"], W["pinned"])]
    want = np.where(got["mask"] == 1, sum(a @ b for a, b in zn), sum(a @ b for a, b in zq))
    l1 = sum(np.abs(a) @ np.abs(b) for a, b in zn + zq)
    bound = 2 * D * 2.0 ** -23 * l1
    assert np.all(np.abs(got["Y_cell"] - want) <= bound)
    assert np.all(got["Y_cell"] >= np.maximum(sum(a @ b for a, b in zn), zq[0][0] @ zq[0][1]) - bound)
    _within(got["Y_net"], [(got["Xs_self"], W["self_pins"]), (got["H_pins"], W["neigh_pins"])], "Y_net", 2 * D)
    # weight gradients
    dZn, dZq = np.where(got["mask"] == 1, dYc, 0.0), np.where(got["mask"] == 0, dYc, 0.0)
    for n, A, B in (("self_near", "Xs_cell", dZn), ("neigh_near", "H_near", dZn), ("pinned", "H_pinned", dZq),
                    ("self_pins", "Xs_self", dYn), ("neigh_pins", "H_pins", dYn)):
        _within(got[n], [(got[A].T, B)], "dW." + n, len(B))
    # input gradients: dZ W^T sampled at the selections, and the transposed relations over dZ W^T

    def dense(r, m, n):
        a = np.zeros((m, n))
        np.add.at(a, (np.repeat(np.arange(m), np.diff(r[0])), r[1]), r[2].astype(np.float64))
        return a
    keep = {u: np.zeros((len(i), D)) for u, i in got["sel"].items()}
    for u, i in got["sel"].items():
        np.put_along_axis(keep[u], i.astype(np.int64), 1.0, axis=1)
    an, ap, aq = dense(near, Nc, Nc), dense(pins, Nn, Nc), dense(pinned, Nc, Nn)

    def grads(absolute):
        g = (lambda x: np.abs(x)) if absolute else (lambda x: x)
        w = {n: g(x) for n, x in W.items()}
        c = keep["near"] * (g(dZn) @ w["self_near"].T + an.T @ (g(dZn) @ w["neigh_near"].T)) + keep["pins"] * (ap.T @ (g(dYn) @ w["neigh_pins"].T))
        n = keep["self"] * (g(dYn) @ w["self_pins"].T) + keep["pinned"] * (aq.T @ (g(dZq) @ w["pinned"].T))
        return c, n
    for name, want, l1 in zip(("dX_cell", "dX_net"), grads(False), grads(True)):
        assert np.all(np.abs(got[name] - want) <= 2 * D * 2.0 ** -23 * l1), name


@pytest.mark.parametrize("rows", [4096, 4097])
def test_products_where_workgroups_get_a_second_chunk(rows):
    """128 and 129 chunks of 32 rows: up to 128, every workgroup of the weight gradients has one chunk."""
    test_products_at_tile_edges(128, 32, 24, 40, rows)


@pytest.mark.parametrize("D", [32, 96, 128])
def test_ends_of_the_range(D):
    """Infinite operands give the infinities and not-a-numbers of the fp32 products, the largest finite numbers stay finite."""
    say(f"dense range D={D}")
    Nc, Nn = 40, 70
    rng = np.random.default_rng(D)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)             # noqa: E731
    W = {n: rng.uniform(0.01, 0.02, (D, D)).astype(np.float32) * np.where(np.arange(D) % 2, 1, -1).astype(np.float32) for n in P.WEIGHT_NAMES}
    X_cell, X_net, dYc, dYn = f(Nc, D), f(Nn, D), f(Nc, D), f(Nn, D)
    big = np.finfo(np.float32).max
    X_net[3, 5], X_net[4, 6], X_net[5, 7], X_net[6, 8] = np.inf, -np.inf, big, -big
    X_cell[0, 1] = np.inf
    dYn[10, 2], dYn[11, 3], dYn[12, 4] = np.inf, big, np.nan
    got = _run(Nc, Nn, D, (D, D, D), rng, X_cell, X_net, W, dYc, dYn, edges=False)
    with np.errstate(invalid="ignore", over="ignore"):
        y = X_net.astype(np.float64) @ W["self_pins"].astype(np.float64)
        dw = X_net.astype(np.float64).T @ dYn.astype(np.float64)
        dx = dYn.astype(np.float64) @ W["self_pins"].astype(np.float64).T
    rows = [3, 4, 5, 6]
    assert np.array_equal(got["Y_net"][3:5], y[3:5]) and np.isinf(y[3:5]).all()
    assert np.allclose(got["Y_net"][5:7], y[5:7], rtol=1e-6, atol=0)
    others = [r for r in range(Nn) if r not in rows]
    assert np.isfinite(got["Y_net"][others]).all()
    assert np.array_equal(got["dX_net"][10], dx[10]) and np.isinf(dx[10]).all()
    assert np.allclose(got["dX_net"][11], dx[11], rtol=1e-6, atol=0) and np.isnan(got["dX_net"][12]).all()
    assert np.isnan(got["self_pins"][:, 4]).all()
    plain = [c for c in range(D) if c not in (2, 3, 4)]
    assert np.array_equal(got["self_pins"][5, plain], dw[5, plain]) and np.isinf(dw[5, plain]).all()
    assert np.isinf(got["Y_cell"][0]).any() and np.isfinite(got["Y_cell"][1:]).all()


def _as_fp32(got, want, what):
    """Single products: infinite where the fp32 product is, with its sign, and close to it elsewhere (a product off the exact
    one by 2^-24, in sums that add zeros only)."""
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf].astype(np.float64)), (what, got[inf][:8], want[inf][:8])
    w = want[~inf].astype(np.float64)
    assert np.all(np.abs(got[~inf] - w) <= 2.0 ** -22 * np.abs(w)), what
    assert inf.any() and (~inf).any()


@pytest.mark.parametrize("D", [32, 64, 96, 128])
def test_overflow_as_in_fp32(D):
    """Products with large factors on either side: an infinite or overflowing product is an infinity of the right sign whatever
    the other factor's lower parts are (their products with the large factor overflow too, to either side), and a product
    just below the largest number is finite."""
    say(f"dense overflow D={D}")
    rng = np.random.default_rng(100 + D)

    def factors(*s):
        x = np.exp2(rng.uniform(-3, 12, s)) * rng.choice([-1.0, 1.0], s)
        x[..., 0], x[..., 1], x[..., 2], x[..., 3] = 1.999, 998.5, -514.9, 1002.5
        return x.astype(np.float32)
    W = {n: factors(D, D) for n in P.WEIGHT_NAMES}
    big = np.array([np.inf, -np.inf, 3e38, -np.finfo(np.float32).max, 1.7e38, -1.7e38, 3.39e38, 1e36, -1e30, 1.0, -1e-30], np.float32)
    # one large entry per row: every output is one product
    n = 4 * len(big) + 1
    vals, at = np.resize(big, n), (np.arange(n) * 7) % D
    X = np.zeros((n, D), np.float32)
    X[np.arange(n), at] = vals
    zero = np.zeros((n, D), np.float32)
    got = _run(n, n, D, (D, D, D), rng, X, X, W, zero, X, edges=False)
    with np.errstate(over="ignore"):
        _as_fp32(got["Y_net"], vals[:, None] * W["self_pins"][at], "Y_net")
        near = vals[:, None] * W["self_near"][at]
        _as_fp32(got["Y_cell"], np.maximum(near, np.float32(0)), "Y_cell")               # the pinned branch is zero
        _as_fp32(got["dX_net"], vals[:, None] * W["self_pins"].T[at], "dX_net")
        # one row of large entries: every entry of the weight gradient is one product
        for row in (0, n // 2, n - 1):
            Xr, dY = np.zeros((n, D), np.float32), np.zeros((n, D), np.float32)
            Xr[row], dY[row] = np.resize(big, D), factors(D)
            got = _run(n, n, D, (D, D, D), rng, zero, Xr, W, zero, dY, edges=False)
            _as_fp32(got["self_pins"], Xr[row][:, None] * dY[row][None, :], "dW large entries")
            got = _run(n, n, D, (D, D, D), rng, zero, dY, W, zero, Xr, edges=False)
            _as_fp32(got["self_pins"], dY[row][:, None] * Xr[row][None, :], "dW large gradients")


@pytest.mark.parametrize("D,k", [(32, 32), (64, 40), (96, 24), (128, 128)])
@pytest.mark.parametrize("rows,sign", [(700, "both"), (700, "one"), (33_331, "one")])
def test_as_accurate_as_fp32(D, k, rows, sign):
    """2-norm errors against fp64 at which a 24-bit product stands out from one that has lost a part.  The products of a split
    that are smallest, x1 y3, x2 y2 and x3 y1, are 2^-18 of the whole each (rms); without one of them the error is 2.4e-6 .. 2.7e-6
    on N(0,1) data and 3.4e-7 .. 3.8e-7 on data of one sign (emulated: K = 128).  A rounding to fp32 costs 2^-25.1 = 2.8e-8 (rms); a projection adds up to 16 partial
    sums of up to 256 terms, each rounded once: 2^-23 = 1.2e-7 leaves a factor of two over what was measured, 4e-8 .. 7e-8.
    Weight gradients on data of one sign add some 130 partial sums per workgroup and round the total once; sums that are cut
    off instead of rounded, or added up in 32 bits at the end, come to 6.5e-8 .. 7.4e-8 there, these to 3e-8."""
    say(f"dense accuracy rows={rows} D={D} {sign}")
    rng = np.random.default_rng(D + rows)

    def f(*s):
        x = rng.standard_normal(s).astype(np.float32)
        return np.abs(x) if sign == "one" else x
    W = {n: (f(D, D) / np.sqrt(D)).astype(np.float32) for n in P.WEIGHT_NAMES}
    X_cell, X_net, dYc, dYn = f(rows, D), f(rows, D), f(rows, D), f(rows, D)
    got, *_ = _run(rows, rows, D, (k, k, k), rng, X_cell, X_net, W, dYc, dYn, dup=True)
    alone = _run(rows, rows, D, (D, D, D), rng, X_cell, X_net, W, dYc, dYn, edges=False, dup=True)      # dX: the self terms and nothing else
    W = {n: w.astype(np.float64) for n, w in W.items()}
    mask = got["mask"] == 1
    dZn, dZq, dYn = np.where(mask, dYc, 0.0).astype(np.float64), np.where(mask, 0.0, dYc).astype(np.float64), dYn.astype(np.float64)
    pairs = dict(
        Y_cell=(got["Y_cell"], np.where(mask, got["Xs_cell"] @ W["self_near"] + got["H_near"] @ W["neigh_near"], got["H_pinned"] @ W["pinned"])),
        Y_net=(got["Y_net"], got["Xs_self"] @ W["self_pins"] + got["H_pins"] @ W["neigh_pins"]),
        dX_net=(alone["dX_net"], dYn @ W["self_pins"].T),
        dX_cell=(alone["dX_cell"], np.where(alone["mask"] == 1, dYc, 0.0).astype(np.float64) @ W["self_near"].T))
    for n, (have, want) in pairs.items():
        err = np.linalg.norm(have - want) / np.linalg.norm(want)
        assert err <= 2.0 ** -23, (n, err)
    for n, A, B in (("self_near", "Xs_cell", dZn), ("neigh_near", "H_near", dZn), ("pinned", "H_pinned", dZq),
                    ("self_pins", "Xs_self", dYn), ("neigh_pins", "H_pins", dYn)):
        want = got[A].T @ B
        err = np.linalg.norm(got[n] - want) / np.linalg.norm(want)
        assert err <= (2.0 ** -24 if sign == "one" else 2.0 ** -23), (n, err)


@pytest.mark.parametrize("D", [32, 64, 96, 128])
@pytest.mark.parametrize("rows", [40, 33_000])
def test_weight_gradients_with_sums_that_are_not_finite(D, rows):
    """Sums that overflow or meet infinities are infinities and not-a-numbers as in fp32; the others of the same workgroup are as
    without.  One chunk per workgroup at 40 rows, several at 33 000.  Entries are compared with fp64 products
    where those stay in range (n * 2^-23 of the L1 norm, as above), with their infinities and not-a-numbers elsewhere."""
    say(f"dense non-finite weight gradients D={D} rows={rows}")
    rng = np.random.default_rng(D + rows)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)             # noqa: E731
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    X_cell, X_net, dYc, dYn = f(rows, D), f(rows, D), f(rows, D), f(rows, D)
    big = np.finfo(np.float32).max
    at = rng.permutation(rows)[:6]
    X_cell[at[0], 3], dYc[at[1], 5], dYc[at[2], 7] = np.inf, -np.inf, np.nan
    X_net[at[3], 4], dYn[at[4], 6], dYn[at[5], 9] = -np.inf, np.inf, np.nan
    X_cell[at[3], 11] = X_net[at[0], 11] = big                           # finite, with parts that round up
    got = _run(rows, rows, D, (D, D, D), rng, X_cell, X_net, W, dYc, dYn, edges=False, dup=True)
    m = got["mask"] == 1
    for name, A, B in (("self_near", X_cell, np.where(m, dYc, np.float32(0))), ("self_pins", X_net, dYn)):
        A, B = A.astype(np.float64), B.astype(np.float64)
        with np.errstate(invalid="ignore", over="ignore"):
            want, l1 = A.T @ B, np.abs(A).T @ np.abs(B)
            off = np.abs(got[name] - want)
        inside = l1 < big
        assert inside.any() and np.isnan(want).any() and np.isinf(want).any()
        assert np.all(off[inside] <= rows * 2.0 ** -23 * l1[inside]), name
        assert np.array_equal(np.isnan(got[name])[~np.isfinite(l1)], np.isnan(want)[~np.isfinite(l1)]), name
        inf = np.isinf(want)
        assert np.array_equal(got[name][inf], want[inf]), name
    assert np.all(got["pinned"][:, [c for c in range(D) if c not in (5, 7)]] == 0)       # H_pinned is zero
