"""The backward's shared launches -- weight gradients beside projections, their partial sums behind the last rows of the transposed
DR-SpMM -- against a launch of its own for every step: the same bits, whatever the widths leave to which launch.  (Small layers, where a
workgroup has one chunk of rows either way, and one of which either side fills the chip; in between the sides share workgroups and the
weight gradients differ by the order of their sums, tests/test_gpu_rows_per_wavefront.py.)"""
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


def test_large_layers_sum_their_weight_gradients_as_in_launches_of_their_own():
    """1.2 M cells and 0.9 M nets of 128: either node type gets as many workgroups as alone, so that no running sum gets longer (and
    less exact) by sharing the launch.  No edges: the gradients of the self terms are what is compared."""
    D, k, Nc, Nn = 128, 32, 1_200_000, 900_000
    say(f"shared launches, large: D={D} {Nc} cells {Nn} nets")
    gen = torch.Generator(device="cuda").manual_seed(5)
    f = lambda *s: torch.randn(*s, device="cuda", generator=gen)         # noqa: E731
    empty = lambda m, n: P.Csr(m, n, torch.zeros(m + 1, dtype=torch.int32, device="cuda"),     # noqa: E731
                               torch.empty(0, dtype=torch.int32, device="cuda"), torch.empty(0, device="cuda"))
    layer = P.HeteroConv(empty(Nc, Nc), empty(Nn, Nc), empty(Nc, Nn), D, k, k)
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    saved = layer.alloc_saved()
    X, dY = (f(Nc, D), f(Nn, D)), (f(Nc, D), f(Nn, D))
    layer.heteroconv_fwd(*X, W, torch.empty_like(X[0]), torch.empty_like(X[1]), saved)

    def backward(mode):
        layer.heteroconv_set_overlap(mode)
        dX = torch.full((Nc, D), float("nan"), device="cuda"), torch.full((Nn, D), float("nan"), device="cuda")
        dW = {n: torch.full((D, D), float("nan"), device="cuda") for n in P.WEIGHT_NAMES}
        layer.heteroconv_bwd(*dY, W, saved, *dX, dW)
        return [*dX] + [dW[n] for n in P.WEIGHT_NAMES]

    apart, shared = backward(P.DR_OVERLAP_OFF), backward(P.DR_OVERLAP_AUTO)
    for a, b in zip(apart, shared):
        assert not torch.isnan(b).any()
        assert torch.equal(a, b)
    layer.heteroconv_destroy()
