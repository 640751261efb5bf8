"""Weight gradients of operands that hold infinities, not-a-numbers and numbers around 2^62, from where on a chunk's small products
are cut to finite numbers: in the gradients, in the selections (in registers and past them) and in the gathered rows."""
import numpy as np
import pytest
import torch

import paper_2508_16769_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


def _layer(rows, D, k, seed):
    """A layer without edges; what its backward reads is put into `saved`."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    f = lambda *s: torch.randn(*s, device="cuda", generator=gen)         # noqa: E731
    empty = P.Csr(rows, rows, torch.zeros(rows + 1, dtype=torch.int32, device="cuda"),
                  torch.empty(0, dtype=torch.int32, device="cuda"), torch.empty(0, device="cuda"))
    layer = P.HeteroConv(empty, empty, empty, D, k, k)
    W, saved = {n: f(D, D) for n in P.WEIGHT_NAMES}, layer.alloc_saved()
    layer.heteroconv_fwd(f(rows, D), f(rows, D), W, f(rows, D), f(rows, D), saved)
    for n in ("H_near", "H_pins", "H_pinned"):
        saved[n].copy_(f(rows, D))
    saved["mask"].copy_(torch.randint(0, 2, (rows, D), dtype=torch.uint8, device="cuda", generator=gen))
    dY, dX = [f(rows, D), f(rows, D)], [f(rows, D), f(rows, D)]
    return layer, W, saved, dY, dX, {n: f(D, D) for n in P.WEIGHT_NAMES}


@pytest.mark.parametrize("rows", [300, 20_000])                          # a chunk per workgroup, several
@pytest.mark.parametrize("D,k", [(32, 8), (64, 40), (96, 24), (128, 32), (128, 128)])
@pytest.mark.parametrize("where", ["dY", "vals", "H"])
def test_operands_that_overflow(where, D, k, rows):
    say(f"wide operands in {where}: rows={rows} D={D} k={k}")
    layer, W, saved, dY, dX, dW = _layer(rows, D, k, D + rows)
    into = dict(dY=dY, vals=[saved["vals_cell"], saved["vals_net"]], H=[saved["H_near"], saved["H_pinned"], saved["H_pins"]])[where]
    big = [float("inf"), float("-inf"), float("nan"), 3e38, -3e38] + [s * 2.0 ** e for s in (1, -1) for e in (61.99, 62, 63, 120)]
    rng = np.random.default_rng(rows + D)
    for t in into:
        for r, v in zip(rng.permutation(rows), big):
            t[int(r), int(rng.integers(t.shape[1]))] = v
    layer.heteroconv_bwd(*dY, W, saved, *dX, dW)
    d, zero = (lambda t: t.double()), torch.zeros((), device="cuda")
    dense = lambda n: torch.zeros(rows, D, device="cuda").scatter_(1, saved["idx_" + n].long(), saved["vals_" + n])      # noqa: E731
    m = saved["mask"] == 1
    near, pinned = torch.where(m, dY[0], zero), torch.where(m, zero, dY[0])
    met = 0
    for n, A, B in (("self_near", dense("cell"), near), ("neigh_near", saved["H_near"], near), ("pinned", saved["H_pinned"], pinned),
                    ("self_pins", dense("net"), dY[1]), ("neigh_pins", saved["H_pins"], dY[1])):
        want, l1 = d(A).T @ d(B), d(A).abs().T @ d(B).abs()
        got = d(dW[n])
        inside = l1 < torch.finfo(torch.float32).max
        assert inside.any(), n
        met += int((~inside).sum())
        # one rounding per product, chunk and partial sum: rows * 2^-23 of the L1 norm bounds them all
        assert bool(((got - want).abs()[inside] <= rows * 2.0 ** -23 * l1[inside]).all()), n
        outside = ~torch.isfinite(l1)                                    # in between the order of the sums decides
        assert torch.equal(torch.isnan(got)[outside], torch.isnan(want)[outside]), n
        assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), n
    assert met
    layer.heteroconv_destroy()


def test_an_infinity_costs_no_second_pass():
    """One infinite gradient among 250 000 rows: the launch that meets it takes about as long as without (a workgroup that summed
    its rows twice made it 1.7 times as long)."""
    rows, D, k = 250_000, 128, 32
    say("time of weight gradients with an infinity")
    layer, W, saved, dY, dX, dW = _layer(rows, D, k, 3)
    layer.heteroconv_profile(True)

    def best():
        times = []
        for _ in range(6):
            layer.heteroconv_bwd(*dY, W, saved, *dX, dW)
            torch.cuda.synchronize()
            times.append([t for n, (t, _) in layer.heteroconv_kernel_times().items() if n.startswith("wgrad")])
        return np.min(np.array(times[1:]), axis=0)
    finite = best()
    for t in dY:
        t[rows // 2, 5] = float("inf")
    infinite = best()
    say(f"weight gradients ms: finite {finite}, one infinity {infinite}")
    assert np.all(infinite < 1.3 * finite)
    layer.heteroconv_destroy()
