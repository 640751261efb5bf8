"""DR-SpMM where its row dispatch changes: the row counts at which a wavefront goes from 8 rows to 16 and 32, and row lengths at
which a row passes from one lane group to a wavefront (32) and to a whole workgroup (256)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_16769_amd as P
from gpu_util import assert_elem_bound, assert_row_bound, dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,D,k", [(33, 32, 8), (1000, 100, 25), (49_152, 64, 16), (49_153, 64, 16), (49_153, 64, 40),
                                   (40_960, 64, 16), (40_961, 64, 16), (102_401, 32, 8)])
def test_row_lengths_at_the_dispatch_edges(M, D, k):
    say(f"spmm rows M={M} D={D} k={k}")
    rng = np.random.default_rng(M + k)
    N = 700
    deg = rng.integers(0, 4, M)
    edge_lengths = [0, 1, 31, 32, 33, 255, 256, 257, 258, 511, 1025, 2000]
    deg[rng.permutation(M)[:len(edge_lengths)]] = edge_lengths
    deg[:2] = 300, 299                                   # two very long rows side by side
    deg[-1] = 1024                                       # one in the last, partly filled block
    rp = np.zeros(M + 1, np.int32)
    np.cumsum(deg, out=rp[1:])
    ci = rng.integers(0, N, int(rp[-1])).astype(np.int32)
    av = rng.uniform(0.05, 1.0, ci.shape[0]).astype(np.float32)
    A = P.Csr(M, N, dev(rp), dev(ci), dev(av))
    # forward: rows are the destinations
    ov, oi = oracle.topk(rng.standard_normal((N, D)).astype(np.float32), k)
    want, l1row, l1elem = oracle.spmm_fwd(rp, ci, av, ov, oi, D, want_l1elem=True)
    H = torch.full((M, D), float("nan"), dtype=torch.float32, device="cuda")
    P.dr_spmm_fwd(A, dev(ov, torch.float32), dev(oi.astype(np.uint16).view(np.int16)), D, k, H)
    assert_row_bound(H.cpu().numpy(), want, l1row, "fwd")
    # at most 2000 terms of at most 2^-24 * (partial sum) each, added in 32 partial sums of at most 63: 1e-5 holds
    assert_elem_bound(H.cpu().numpy(), want, l1elem, "fwd")
    # backward: the same rows as sources
    oi2 = np.sort(np.argsort(rng.random((M, D)), axis=1)[:, :k], axis=1).astype(np.int32)
    dH = rng.standard_normal((N, D)).astype(np.float32)
    want, l1row, l1elem = oracle.spmm_bwd(rp, ci, av, dH, oi2, want_l1elem=True)
    G = torch.full((M, k), float("nan"), dtype=torch.float32, device="cuda")
    P.dr_spmm_bwd(A, dev(dH), dev(oi2.astype(np.uint16).view(np.int16)), D, k, G)
    assert_row_bound(G.cpu().numpy(), want, l1row, "bwd")
    assert_elem_bound(G.cpu().numpy(), want, l1elem, "bwd")


@pytest.mark.parametrize("k", [1, 4, 7, 9, 12, 15, 16, 17, 23, 24, 25, 31, 32])
def test_forward_pairs_at_any_alignment(k):
    """Widths that fill no vector, in arrays that start one element past an aligned address, with NaN on either side."""
    M, N, D = 37, 29, 68
    say(f"spmm pairs k={k}")
    rng = np.random.default_rng(k)
    rp = np.arange(M + 1, dtype=np.int32) * 6
    ci = rng.integers(0, N, 6 * M).astype(np.int32)
    ci[:2] = 0, N - 1                                    # the first and the last row of the arrays
    av = rng.uniform(0.05, 1.0, 6 * M).astype(np.float32)
    ov, oi = oracle.topk(rng.standard_normal((N, D)).astype(np.float32), k)
    vals = torch.full((N * k + 2,), float("nan"), dtype=torch.float32, device="cuda")
    idx = torch.zeros(N * k + 2, dtype=torch.int16, device="cuda")
    vals[1:-1] = dev(ov, torch.float32).flatten()
    idx[1:-1] = dev(oi.astype(np.uint16).view(np.int16)).flatten()
    want, _, l1elem = oracle.spmm_fwd(rp, ci, av, ov, oi, D, want_l1elem=True)
    H = torch.full((M, D), float("nan"), dtype=torch.float32, device="cuda")
    P.dr_spmm_fwd(P.Csr(M, N, dev(rp), dev(ci), dev(av)), vals[1:-1].view(N, k), idx[1:-1].view(N, k), D, k, H)
    assert_elem_bound(H.cpu().numpy(), want, l1elem, "fwd")
