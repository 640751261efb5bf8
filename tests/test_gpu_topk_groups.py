"""D-ReLU where several rows share a wavefront (up to 128 columns, whole float4s) and at the edges of that path: partly filled
lane groups and wavefronts, rows of the second and later trips, and rows that its guided search has no guess for (ties,
constant rows, infinities, scales that jump from row to row).  Exact: selections and values are compared bit for bit."""
import numpy as np
import pytest
import torch

import paper_2508_16769_amd as P
from gpu_util import dev, host_idx, say

pytestmark = pytest.mark.gpu


def _expected(X, k):
    """k largest per row, ties to the lowest column, ascending columns (-0 ties with +0)."""
    order = np.argsort(-(X + np.float32(0)), axis=1, kind="stable")[:, :k]
    cols = np.sort(order, axis=1)
    return np.take_along_axis(X, cols, axis=1), cols.astype(np.int32)


def _rows(rng, n, D, kind):
    X = rng.standard_normal((n, D)).astype(np.float32)
    if kind == "ties":
        X = np.round(X * 2).astype(np.float32) / 2
        X[X == 0] = rng.choice(np.array([0.0, -0.0], np.float32), int((X == 0).sum()))
    elif kind == "skewed":
        X = np.where(X > 2, X * 1e6, np.exp(2 * X)).astype(np.float32)
    elif kind == "hard":
        X *= np.exp2(rng.integers(-120, 120, (n, 1))).astype(np.float32)       # every row another scale, denormals among them
        X[::7] = 3.0                                                          # constant rows
        X[1::7] = np.where(rng.random((len(X[1::7]), D)) < 0.9, 0.0, X[1::7])
        X[2::7, 0] = np.inf
        X[2::7, D // 2] = -np.inf
        X[3::7] = np.inf * np.sign(X[3::7])
    return X


@pytest.mark.parametrize("kind", ["normal", "ties", "skewed", "hard"])
@pytest.mark.parametrize("D", [4, 32, 36, 64, 68, 96, 100, 128, 132])
def test_selection_at_the_edges_of_the_lane_groups(D, kind):
    rng = np.random.default_rng(D)
    for n in (1, 15, 16, 17, 131, 1000):
        for k in sorted({1, 3, D // 4 + 1, D // 2, D - 1, D}):
            if k < 1:
                continue
            say(f"topk groups D={D} n={n} k={k} {kind}")
            X = _rows(rng, n, D, kind)
            wv, wi = _expected(X, k)
            vals = torch.full((n, k), float("nan"), device="cuda")
            idx = torch.full((n, k), -1, dtype=torch.int16, device="cuda")
            P.dr_topk(dev(X), k, vals, idx)
            assert np.array_equal(host_idx(idx), wi)
            assert np.array_equal(vals.cpu().numpy().view(np.uint32), wv.view(np.uint32))


@pytest.mark.parametrize("n,D,k", [(300_011, 32, 8), (150_001, 64, 16), (140_003, 96, 24), (140_003, 128, 32)])
def test_later_trips_of_a_wavefront(n, D, k):
    say(f"topk groups n={n} D={D} k={k}")
    X = _rows(np.random.default_rng(n), n, D, "normal")
    X[n // 2:] *= 1000.0                                    # rows of another scale in the same launch
    wv, wi = _expected(X, k)
    vals, idx = torch.empty((n, k), device="cuda"), torch.empty((n, k), dtype=torch.int16, device="cuda")
    P.dr_topk(dev(X), k, vals, idx)
    assert np.array_equal(host_idx(idx), wi)
    assert np.array_equal(vals.cpu().numpy(), wv)


@pytest.mark.parametrize("D,k", [(64, 7), (128, 32)])
def test_alignment_of_inputs_and_outputs(D, k):
    """Inputs that take no float4 loads go the general way; outputs that take no wide stores are written one by one."""
    say(f"topk alignment D={D} k={k}")
    n = 1003
    X = _rows(np.random.default_rng(k), n, D, "normal")
    wv, wi = _expected(X, k)
    for shift_in, shift_v, shift_i in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 1, 3)):
        buf = torch.empty(n * D + 4, device="cuda")
        x = buf[shift_in:shift_in + n * D].view(n, D)
        x.copy_(dev(X))
        vb, ib = torch.full((n * k + 8,), 7.0, device="cuda"), torch.full((n * k + 8,), 7, dtype=torch.int16, device="cuda")
        vals, idx = vb[shift_v:shift_v + n * k].view(n, k), ib[shift_i:shift_i + n * k].view(n, k)
        P.dr_topk(x, k, vals, idx)
        assert np.array_equal(host_idx(idx), wi) and np.array_equal(vals.cpu().numpy(), wv)
        assert bool((vb[shift_v + n * k:] == 7).all()) and bool((vb[:shift_v] == 7).all())
        assert bool((ib[shift_i + n * k:] == 7).all()) and bool((ib[:shift_i] == 7).all())


@pytest.mark.parametrize("n", [67, 33_003])
@pytest.mark.parametrize("D", [32, 36, 64, 100, 128])
def test_not_a_number_rows_stay_to_themselves(D, n):
    """Memory filled with 0xFF, and other not-a-numbers whose keys are the ends of the key range, beside ordinary rows: those
    are exact, and every row keeps k columns of its own (positive not-a-numbers above all, negative ones below all)."""
    rng = np.random.default_rng(D + n)
    for k in (1, D // 4, D):
        say(f"topk not-a-numbers D={D} n={n} k={k}")
        X = _rows(rng, n, D, "normal")
        u = X.view(np.uint32)
        u[1::5] = 0xffffffff
        part = rng.random((len(u[2::5]), D)) < rng.random((len(u[2::5]), 1))
        u[2::5][part] = 0xffffffff
        u[3::10] = 0x7fffffff
        u[8::10] = rng.choice(np.array([0xffffffff, 0x7fffffff, 0xfffffffe, 0x7f800000, 0], np.uint32), u[8::10].shape)
        plain = np.where(X == 0, np.uint32(0), u)
        key = np.where(plain >> 31 != 0, ~plain, plain | np.uint32(0x80000000)).astype(np.int64)
        cols = np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1)
        vals = torch.full((n, k), 7.0, device="cuda")
        idx = torch.full((n, k), -1, dtype=torch.int16, device="cuda")
        P.dr_topk(dev(X), k, vals, idx)
        assert np.array_equal(host_idx(idx), cols)
        assert np.array_equal(vals.cpu().numpy().view(np.uint32), np.take_along_axis(u, cols, axis=1))


def _check_on_gpu(X, k, vals, idx):
    """Against torch's stable sort of the whole rows (finite or infinite values; -0 ties with +0)."""
    cols = torch.sort(-(X + 0.0), dim=1, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx.to(torch.int64), cols)
    assert torch.equal(vals.view(torch.int32), torch.gather(X, 1, cols).view(torch.int32))


@pytest.mark.parametrize("n,D,k", [(280_003, 64, 8), (140_003, 100, 25), (210_011, 128, 32)])
def test_trips_that_follow_a_trace(n, D, k):
    """Rows no guess from their moments serves, for two and more trips of a wavefront; then rows of another law and scale."""
    say(f"topk trace n={n} D={D} k={k}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    X = torch.rand((n, D), device="cuda", generator=gen)
    big = torch.rand((n, D), device="cuda", generator=gen) < 0.02
    X = torch.where(big, 1e6 * torch.randn((n, D), device="cuda", generator=gen), X)
    X[-n // 4:] = torch.exp(3 * torch.randn((n // 4 + 1, D), device="cuda", generator=gen))
    X[-n // 8:] *= 1e-6
    X[::11] = torch.round(4 * X[::11])
    vals, idx = torch.empty((n, k), device="cuda"), torch.empty((n, k), dtype=torch.int16, device="cuda")
    P.dr_topk(X, k, vals, idx)
    _check_on_gpu(X, k, vals, idx)


@pytest.mark.parametrize("kind", ["normal", "ties", "skewed", "hard"])
@pytest.mark.parametrize("D", [4, 32, 36, 64, 68, 96, 100, 128])
def test_selection_where_fewer_lanes_share_a_row(D, kind):
    """From 32768 rows on a row has 4 or 8 lanes; rows that are no whole number of wavefronts, widths that leave lanes without a
    column, outputs that take no wide stores."""
    rng = np.random.default_rng(1000 + D)
    for n, shift in ((32_768, 0), (33_003, 1)):
        X = dev(_rows(rng, n, D, kind))
        for k in sorted({1, D // 4 + 1, D}):
            say(f"topk lanes D={D} n={n} k={k} {kind}")
            vb, ib = torch.full((n * k + 8,), 7.0, device="cuda"), torch.full((n * k + 8,), 7, dtype=torch.int16, device="cuda")
            vals, idx = vb[shift:shift + n * k].view(n, k), ib[shift:shift + n * k].view(n, k)
            P.dr_topk(X, k, vals, idx)
            _check_on_gpu(X, k, vals, idx)
            assert bool((vb[shift + n * k:] == 7).all()) and bool((vb[:shift] == 7).all())
            assert bool((ib[shift + n * k:] == 7).all()) and bool((ib[:shift] == 7).all())


@pytest.mark.parametrize("Nc,Nn", [(1_500, 1_001), (30_011, 20_003)])
@pytest.mark.parametrize("D,ks", [(32, (8, 3, 5)), (64, (16, 7, 24)), (96, (24, 40, 9)), (128, (32, 12, 64))])
def test_two_selections_of_tied_rows(D, ks, Nc, Nn):
    """A layer with a width per relation selects twice from every row; clearing the keys that lose a tie in the first selection must
    not reach the second."""
    say(f"topk twice D={D} ks={ks} Nc={Nc}")
    rng = np.random.default_rng(D + Nc)

    def relation(M, N):
        rowptr = np.arange(M + 1, dtype=np.int32)
        return P.Csr(M, N, dev(rowptr), dev(rng.integers(0, N, M).astype(np.int32)), torch.ones(M, device="cuda"))

    layer = P.HeteroConv(relation(Nc, Nc), relation(Nn, Nc), relation(Nc, Nn), D, per_relation=ks)
    saved = layer.alloc_saved()
    W = {n: torch.zeros((D, D), device="cuda") for n in P.WEIGHT_NAMES}
    X = {"cell": dev(_rows(rng, Nc, D, "ties")), "net": dev(_rows(rng, Nn, D, "hard"))}
    X["net"][1::3] = dev(_rows(rng, Nn, D, "ties"))[1::3]
    layer.heteroconv_fwd(X["cell"], X["net"], W, torch.empty((Nc, D), device="cuda"), torch.empty((Nn, D), device="cuda"), saved)
    for name, t, k in (("cell", "cell", ks[0]), ("cell_pins", "cell", ks[1]), ("net", "net", ks[2]), ("net_self", "net", ks[1])):
        _check_on_gpu(X[t], k, saved["vals_" + name], saved["idx_" + name])
    layer.heteroconv_destroy()
