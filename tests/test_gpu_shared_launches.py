"""The backward's shared launches -- weight gradients beside projections, their partial sums behind the last rows of the transposed
DR-SpMM -- against a launch of its own for every step: the same bits, whatever the widths leave to which launch."""
import numpy as np
import pytest
import torch

import paper_2508_16769_amd as P
from gpu_util import dev, random_csr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,ks", [(32, (4, 4, 4)), (64, (16, 16, 16)), (96, (24, 12, 8)), (128, (32, 32, 32)),
                                  (128, (70, 70, 16)), (128, (100, 16, 80))])      # 70 and more: sums that no dense launch takes
@pytest.mark.parametrize("Nc,Nn", [(1, 1), (33, 700), (2048, 1), (3000, 2100), (600, 0)])
def test_shared_launches_give_the_bits_of_separate_ones(D, ks, Nc, Nn):
    say(f"shared launches D={D} k={ks} {Nc} cells {Nn} nets")
    rng = np.random.default_rng(D + Nc)
    f = lambda *s: dev(rng.standard_normal(s).astype(np.float32))        # noqa: E731
    edges = 4 if Nn else 0
    rel = [P.Csr(m, n, *(dev(a) for a in random_csr(rng, m, n, e, dup=True)))
           for m, n, e in ((Nc, Nc, 6), (Nn, Nc, edges), (Nc, Nn or 1, edges))]
    rel[2] = P.Csr(Nc, Nn, rel[2].rowptr, rel[2].colidx, rel[2].vals)
    layer = P.HeteroConv(*rel, D, per_relation=ks)
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    X_cell, X_net, dY_cell, dY_net = f(Nc, D), f(Nn, D), f(Nc, D), f(Nn, D)
    pad = [t if t.numel() else torch.zeros(4, device="cuda") for t in (X_net, dY_net)]      # a pointer for what is empty

    def run(mode):
        layer.heteroconv_set_overlap(mode)
        saved = {n: t if t.numel() else torch.zeros(16, dtype=t.dtype, device="cuda") for n, t in layer.alloc_saved().items()}
        nan = lambda *s: torch.full(s, float("nan"), device="cuda")      # noqa: E731
        Y, dX = (nan(Nc, D), nan(max(Nn, 1), D)), (nan(Nc, D), nan(max(Nn, 1), D))
        dW = {n: nan(D, D) for n in P.WEIGHT_NAMES}
        layer.heteroconv_fwd(X_cell, pad[0], W, *Y, saved)
        layer.heteroconv_bwd(dY_cell, pad[1], W, saved, *dX, dW)
        torch.cuda.synchronize()
        return [Y[0], Y[1][:Nn], dX[0], dX[1][:Nn]] + [dW[n] for n in P.WEIGHT_NAMES]

    apart, shared = run(P.DR_OVERLAP_OFF), run(P.DR_OVERLAP_ON)
    for a, b in zip(apart, shared):
        assert not torch.isnan(b).any()
        assert torch.equal(a, b)
    layer.heteroconv_destroy()
