"""DR-SpMM on both sides of the row counts where a wavefront's share of the rows changes (8, 16 or 32): 40 960 rows, 49 152 where
there are fewer rows than columns, 81 920 for forward rows of a few edges, 2^19."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
import paper_2508_16769_amd as P
from gpu_util import dev, random_csr, say

pytestmark = pytest.mark.gpu

# rows, columns, most edges of a row
SHAPES = [(40_960, 3_000, 11), (40_961, 3_000, 11), (49_152, 50_001, 5), (49_153, 50_001, 5), (81_921, 900, 3), (82_017, 900, 14),
          (524_289, 70, 12)]


@pytest.mark.parametrize("M,N,deg", SHAPES)
@pytest.mark.parametrize("D,k", [(32, 8), (64, 25), (128, 32)])
def test_rows_per_wavefront(M, N, deg, D, k):
    if M > 100_000 and D > 32:
        pytest.skip("the oracle's product of half a million rows is made at one width")
    say(f"rows per wavefront {M} x {N}, D={D} k={k}")
    rng = np.random.default_rng(M + D)
    hub = rng.integers(0, M, 3)
    rowptr, colidx, vals = random_csr(rng, M, N, deg, dup=True, evil_rows=hub, evil_deg=700)
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
