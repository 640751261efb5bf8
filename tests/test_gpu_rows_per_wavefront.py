"""DR-SpMM on both sides of the row counts where a wavefront's share of the rows changes (8, 16 or 32), which depend on edges per row,
on whether there are fewer rows than columns (nets) and on D; the dense backward of a layer likewise."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
import paper_2508_16769_amd as P
from gpu_util import dev, random_csr, say

pytestmark = pytest.mark.gpu

# rows, columns, most edges of a row, bounds of edges per row (20 % of the rows are empty)
SHAPES = [(40_960, 3_000, 11, 0, 9), (40_961, 3_000, 11, 0, 9), (49_152, 50_001, 5, 0, 6), (49_153, 50_001, 5, 0, 6),
          (81_920, 900, 14, 0, 9), (81_921, 900, 14, 0, 9), (81_921, 900, 3, 0, 9), (82_017, 900, 14, 0, 9),
          (81_921, 900, 28, 9, 99), (81_921, 90_000, 5, 0, 6), (90_000, 99_000, 18, 6, 99)]
LARGE = [(102_400, 800, 8, 0, 6), (102_401, 800, 8, 0, 6), (102_401, 800, 18, 6, 9), (163_840, 170_000, 5, 0, 6), (163_841, 170_000, 5, 0, 6),
         (524_288, 70, 28, 9, 99), (524_289, 70, 28, 9, 99), (524_289, 70, 12, 0, 6)]
CASES = [(s, w) for s in SHAPES for w in ((32, 8), (64, 25), (128, 32))] + [(s, w) for s in LARGE for w in ((32, 8), (32, 16))] + [(LARGE[5], (64, 25))]
CASES += [((M, 900, 8, 0, 9), (256, 32)) for M in (49_152, 49_153)]      # wide rows: fewer wavefronts resident


@pytest.mark.parametrize("shape,width", CASES, ids=[f"{s[0]}x{s[1]}_deg{s[2]}_D{w[0]}_k{w[1]}" for s, w in CASES])
def test_rows_per_wavefront(shape, width):
    (M, N, deg, least, most), (D, k) = shape, width
    say(f"rows per wavefront {M} x {N}, D={D} k={k}")
    rng = np.random.default_rng(M + D)
    hub = rng.integers(0, M, 3)
    rowptr, colidx, vals = random_csr(rng, M, N, deg, dup=True, evil_rows=hub, evil_deg=700)
    assert least * M <= len(colidx) < most * M
    X = rng.standard_normal((N, D)).astype(np.float32)
    v, i = oracle.topk(X, k)
    Xs = oracle.densify(v, i, D).astype(np.float64)
    A = sp.csr_matrix((vals.astype(np.float64), colidx, rowptr), shape=(M, N))
    A_dev = P.Csr(M, N, dev(rowptr), dev(colidx), dev(vals))
    v_dev, i_dev = dev(np.asarray(v, np.float32)), dev(np.asarray(i).astype(np.uint16).view(np.int16))
    H = torch.full((M, D), float("nan"), device="cuda")
    P.dr_spmm_fwd(A_dev, v_dev, i_dev, D, k, H)
    got = H.cpu().numpy()
    assert np.all(np.abs(got - A @ Xs) <= 1e-5 * (abs(A) @ np.abs(Xs)))
    # the same pattern as a transposed relation: rows are the sources
    Y = rng.standard_normal((N, D)).astype(np.float32)
    sel = np.sort(rng.permuted(np.tile(np.arange(D, dtype=np.uint16), (M, 1)), axis=1)[:, :k], axis=1)
    G = torch.full((M, k), float("nan"), device="cuda")
    P.dr_spmm_bwd(A_dev, dev(Y), dev(sel.view(np.int16)), D, k, G)
    pick = sel.astype(np.int64)
    want, l1 = A @ Y.astype(np.float64), abs(A) @ np.abs(Y.astype(np.float64))
    assert np.all(np.abs(G.cpu().numpy() - np.take_along_axis(want, pick, 1)) <= 1e-5 * np.take_along_axis(l1, pick, 1))


@pytest.mark.parametrize("D,Nc,Nn", [(64, 60_000, 40_000), (32, 200_000, 62_144), (32, 200_000, 62_145), (64, 300_000, 224_289),
                                     (96, 524_200, 300), (96, 524_300, 300)])
def test_dense_backward(D, Nc, Nn):
    """A layer's input gradients do not depend on how its launches are cut: cells and nets together (8192 D rows in all and 2^19 of
    either are where wavefronts go from 16 rows to 32) against a launch for each, the same bits.  The weight gradients are summed over
    other workgroups and by the last workgroups of the one launch: either way within 4e-7 of fp64 (2-norm), so 2^-20 apart at most."""
    k = 8
    say(f"rows per wavefront, dense: D={D} {Nc} cells {Nn} nets")
    rng = np.random.default_rng(Nc + Nn)
    gen = torch.Generator(device="cuda").manual_seed(D)
    f = lambda *s: torch.randn(*s, device="cuda", generator=gen)         # noqa: E731
    rel = [P.Csr(m, n, *(dev(a) for a in random_csr(rng, m, n, e, dup=True)))
           for m, n, e in ((Nc, Nc, 9), (Nn, Nc, 7), (Nc, Nn, 7))]
    layer = P.HeteroConv(*rel, D, k, k)
    W, saved = {n: f(D, D) for n in P.WEIGHT_NAMES}, layer.alloc_saved()
    layer.heteroconv_fwd(f(Nc, D), f(Nn, D), W, f(Nc, D), f(Nn, D), saved)
    dY = f(Nc, D), f(Nn, D)

    def backward(mode):
        layer.heteroconv_set_overlap(mode)
        dX = torch.full((Nc, D), float("nan"), device="cuda"), torch.full((Nn, D), float("nan"), device="cuda")
        dW = {n: torch.full((D, D), float("nan"), device="cuda") for n in P.WEIGHT_NAMES}
        layer.heteroconv_bwd(*dY, W, saved, *dX, dW)
        return dX, dW

    (a, wa), (b, wb) = backward(P.DR_OVERLAP_OFF), backward(P.DR_OVERLAP_ON)
    for x, y in zip(a, b):
        assert not torch.isnan(y).any() and torch.equal(x, y)
    for n in P.WEIGHT_NAMES:
        assert float((wa[n].double() - wb[n].double()).norm()) <= 2.0 ** -20 * float(wa[n].double().norm()), n
    layer.heteroconv_destroy()
