"""Backward passes of one context on several streams: its scratch is one for all of them, so they have to follow one another
whatever streams the caller uses, without the caller's help."""
import numpy as np
import pytest
import torch

import paper_2508_16769_amd as P
from gpu_util import dev, random_csr, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [P.DR_OVERLAP_AUTO, P.DR_OVERLAP_OFF])
def test_backward_passes_on_alternating_streams(mode):
    Nc, Nn, D, k, passes = 30_000, 20_000, 64, 16, 6
    say(f"streams mode={mode}")
    rng = np.random.default_rng(mode)
    rel = [P.Csr(m, n, *(dev(a) for a in random_csr(rng, m, n, 8, dup=True))) for m, n in ((Nc, Nc), (Nn, Nc), (Nc, Nn))]
    layer = P.HeteroConv(*rel, D, k, k)
    layer.heteroconv_set_overlap(mode)
    f = lambda *s: torch.randn(s, device="cuda")                                 # noqa: E731
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    saved = layer.alloc_saved()
    layer.heteroconv_fwd(f(Nc, D), f(Nn, D), W, f(Nc, D), f(Nn, D), saved)
    dY = [(f(Nc, D), f(Nn, D)) for _ in range(passes)]
    side = [torch.cuda.Stream(), torch.cuda.Stream()]

    def run(streams):
        out = [(f(Nc, D), f(Nn, D), {n: f(D, D) for n in P.WEIGHT_NAMES}) for _ in range(passes)]
        torch.cuda.synchronize()
        for i, ((dc, dn), (xc, xn, dW)) in enumerate(zip(dY, out)):
            layer.heteroconv_bwd(dc, dn, W, saved, xc, xn, dW, stream=streams[i % len(streams)])
        torch.cuda.synchronize()
        return out
    want = run([None])
    for streams in (side, [side[0], None, side[1]]):
        for i, (a, b) in enumerate(zip(run(streams), want)):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), i
            assert all(torch.equal(a[2][n], b[2][n]) for n in P.WEIGHT_NAMES), i
    # the context outlives neither the streams' work nor the event another context may still refer to
    layer.heteroconv_destroy()


def test_contexts_of_one_model_by_themselves_afterwards():
    """Contexts that took part in a training step together, then one of them on a stream of its own, then the first destroyed."""
    Nc, Nn, D, k = 3_000, 2_000, 64, 16
    rng = np.random.default_rng(3)
    graphs = []
    for _ in range(3):
        rel = [P.Csr(m, n, *(dev(a) for a in random_csr(rng, m, n, 6, dup=True))) for m, n in ((Nc, Nc), (Nn, Nc), (Nc, Nn))]
        graphs.append(P.HeteroConv(*rel, D, k, k))
    f = lambda *s: torch.randn(s, device="cuda")                                 # noqa: E731
    g = graphs[1]
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    saved, dYc, dYn = g.alloc_saved(), f(Nc, D), f(Nn, D)
    g.heteroconv_fwd(f(Nc, D), f(Nn, D), W, f(Nc, D), f(Nn, D), saved)

    def bwd(stream):
        dX, dW = (f(Nc, D), f(Nn, D)), {n: f(D, D) for n in P.WEIGHT_NAMES}
        torch.cuda.current_stream().synchronize()
        g.heteroconv_bwd(dYc, dYn, W, saved, *dX, dW, stream=stream)
        return [*dX, *dW.values()]
    want = bwd(None)
    torch.cuda.synchronize()
    model = P.Hgnn(graphs, 2, batched=False)
    theta = f(P.hgnn_num_params(2, D)) * 0.1
    m, v, grad, loss = torch.zeros_like(theta), torch.zeros_like(theta), torch.zeros_like(theta), torch.zeros(1, device="cuda")
    X, Xn, tg = [f(Nc, D) for _ in graphs], [f(Nn, D) for _ in graphs], [f(Nc) for _ in graphs]
    side = torch.cuda.Stream()
    for step in range(1, 4):
        model.hgnn_train_step(X, Xn, tg, theta, m, v, 1e-3, 0.9, 0.999, 1e-8, 0.0, step, grad, loss)
        got = bwd(side)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)), step
    model.hgnn_destroy()
    graphs[0].heteroconv_destroy()
    assert all(torch.equal(a, b) for a, b in zip(bwd(None), want))
    torch.cuda.synchronize()


def test_a_stream_that_was_destroyed_since_the_last_pass():
    import ctypes
    from paper_2508_16769_amd import binding
    Nc, Nn, D, k = 2_000, 1_500, 32, 8
    rng = np.random.default_rng(9)
    rel = [P.Csr(m, n, *(dev(a) for a in random_csr(rng, m, n, 6, dup=True))) for m, n in ((Nc, Nc), (Nn, Nc), (Nc, Nn))]
    layer = P.HeteroConv(*rel, D, k, k)
    f = lambda *s: torch.randn(s, device="cuda")                                 # noqa: E731
    W = {n: f(D, D) for n in P.WEIGHT_NAMES}
    saved, dYc, dYn = layer.alloc_saved(), f(Nc, D), f(Nn, D)
    layer.heteroconv_fwd(f(Nc, D), f(Nn, D), W, f(Nc, D), f(Nn, D), saved)
    torch.cuda.synchronize()

    def bwd(stream):
        out = [f(Nc, D), f(Nn, D)], {n: f(D, D) for n in P.WEIGHT_NAMES}
        torch.cuda.synchronize()
        layer.heteroconv_bwd(dYc, dYn, W, saved, *out[0], out[1], stream=stream)
        return [*out[0], *out[1].values()]
    hip = binding.hip_runtime()
    own = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(own), 1) == 0
    first = bwd(own.value)
    assert hip.hipStreamSynchronize(own) == 0 and hip.hipStreamDestroy(own) == 0
    second = bwd(None)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(first, second))
    layer.heteroconv_destroy()
