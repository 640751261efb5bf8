"""Stable transpose and edge values at the sizes where the column partition changes shape: bucket and tile edges, runs of
empty rows longer than a wavefront, one column that holds everything, more columns than one bucket's workgroup owns."""
import numpy as np
import pytest

import oracle
from gpu_util import say

pytestmark = pytest.mark.gpu


def _pattern(rng, M, N, E, law):
    """CSR pattern with E entries; integers only, so the comparison is exact."""
    if law == "one_row":
        rows = np.full(E, M // 2)
    elif law == "tail_rows":                      # long runs of empty rows in front of and between the rows that hold entries
        rows = rng.choice(np.array([0, M // 3, M - 1]), E)
    else:
        rows = rng.integers(0, M, E)
    cols = np.full(E, N - 1) if law == "one_col" else rng.integers(0, N, E)
    if law == "skewed_cols":                      # half of all entries in 3 columns
        hot = rng.random(E) < 0.5
        cols[hot] = rng.choice(np.array([0, N // 2, N - 1]), int(hot.sum()))
    rows = np.sort(rows, kind="stable")
    rp = np.zeros(M + 1, np.int32)
    np.cumsum(np.bincount(rows, minlength=M), out=rp[1:])
    return rp, cols.astype(np.int32)


@pytest.mark.parametrize("M,N,E,law", [
    (1, 1, 1, "uniform"), (3, 64, 63, "uniform"), (3, 65, 65, "uniform"), (700, 4096, 4095, "uniform"),
    (700, 4097, 4097, "skewed_cols"), (5000, 1, 3000, "uniform"), (5000, 333, 9000, "tail_rows"), (1, 90_000, 8193, "one_row"),
    (40_000, 65_537, 300_001, "skewed_cols"), (9_000, 2_000, 70_000, "one_col"), (100_000, 1_300_000, 2_100_000, "uniform"),
    (60_000, 2_200_001, 400_000, "skewed_cols"),
    # the line between counting columns with atomics and by the partition
    (90_000, 70_000, 1 << 19, "skewed_cols"), (90_000, 70_000, (1 << 19) + 1, "skewed_cols"), (60_000, 2_200_001, 600_000, "skewed_cols"),
])
def test_transpose_and_values_exact(M, N, E, law):
    import torch
    import paper_2508_16769_amd as P
    say(f"setup M={M} N={N} E={E} {law}")
    rng = np.random.default_rng(M + 7 * N + 11 * E)
    rp, ci = _pattern(rng, M, N, E, law)
    d_rp, d_ci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    deg_in, deg_out = np.diff(rp).astype(np.float64), np.bincount(ci, minlength=N).astype(np.float64)
    rows = np.repeat(np.arange(M), np.diff(rp))
    for mode in (P.DR_NORM_MEAN, P.DR_NORM_SYM):
        vals = torch.empty(E, dtype=torch.float32, device="cuda")
        ws = torch.empty(max(256, P.dr_csr_normalize_workspace_bytes(mode, M, N, E)), dtype=torch.uint8, device="cuda")
        P.dr_csr_normalize(mode, M, N, d_rp, d_ci, vals, ws)
        want = 1.0 / deg_in[rows] if mode == P.DR_NORM_MEAN else 1.0 / np.sqrt(deg_in[rows] * deg_out[ci])
        assert np.array_equal(vals.cpu().numpy(), want.astype(np.float32))
    ids = torch.arange(E, dtype=torch.int32, device="cuda").view(torch.float32)      # the values name the entries
    At = P.device_transpose(P.Csr(M, N, d_rp, d_ci, ids))
    t_rp, t_ci, _ = oracle.csr_transpose(M, N, rp, ci, np.ones(E, np.float64))
    assert np.array_equal(At.rowptr.cpu().numpy(), t_rp)
    assert np.array_equal(At.colidx.cpu().numpy(), t_ci)
    assert np.array_equal(At.vals.view(torch.int32).cpu().numpy(), np.argsort(ci, kind="stable"))


def test_gaps_of_empty_rows_cost_little():
    """Entries on either side of 2^26 empty rows, and entries a few hundred or some thousand empty rows apart: exact results,
    and no wavefront walks a gap row by row (64 rows per 0.4 us would take this call 0.4 s; it takes well below 1 ms)."""
    import torch
    import paper_2508_16769_amd as P
    M, N = (1 << 26) + 5000, 97
    deg = torch.zeros(M, dtype=torch.int64)
    deg[0], deg[1], deg[M - 1] = 40, 1, 700
    deg[2:600:7] = 3
    deg[1000:3000:260], deg[M - 5000:M - 100:331] = 2, 1              # just past the windows that are walked before a search
    rp = torch.zeros(M + 1, dtype=torch.int64)
    rp[1:] = torch.cumsum(deg, 0)
    E = int(rp[-1])
    say(f"setup gaps M={M} E={E}")
    rows = torch.repeat_interleave(torch.arange(M), deg).numpy()
    rng = np.random.default_rng(5)
    ci = rng.integers(0, N, E).astype(np.int32)
    d_rp, d_ci = rp.to(torch.int32).cuda(), torch.from_numpy(ci).cuda()
    vals = torch.empty(E, device="cuda")
    P.dr_csr_normalize(P.DR_NORM_MEAN, M, N, d_rp, d_ci, vals, None)
    assert np.array_equal(vals.cpu().numpy(), (1.0 / deg.numpy()[rows]).astype(np.float32))
    ids = torch.arange(E, dtype=torch.int32, device="cuda").view(torch.float32)
    A = P.Csr(M, N, d_rp, d_ci, ids)
    At = P.device_transpose(A)
    order = np.argsort(ci, kind="stable")
    assert np.array_equal(At.vals.view(torch.int32).cpu().numpy(), order)
    assert np.array_equal(At.colidx.cpu().numpy(), rows[order])
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    P.dr_csr_normalize(P.DR_NORM_MEAN, M, N, d_rp, d_ci, vals, None)
    stop.record()
    torch.cuda.synchronize()
    assert start.elapsed_time(stop) < 50.0


def test_as_many_entries_as_accepted():
    """2^31 - 1 entries, the most a relation may have: entry e sits in row e // d and column e % N, so every result is known
    in closed form and compared in full, piece by piece."""
    import torch
    import paper_2508_16769_amd as P
    E, N, d = 2 ** 31 - 1, 1_000_003, 21_475
    M = -(-E // d)
    say(f"setup M={M} N={N} E={E}")
    dev, step = "cuda", 1 << 26
    rp = torch.clamp(torch.arange(M + 1, dtype=torch.int64, device=dev) * d, max=E).to(torch.int32)
    ci = torch.empty(E, dtype=torch.int32, device=dev)
    ids = torch.empty(E, dtype=torch.int32, device=dev)
    for s in range(0, E, step):
        e = torch.arange(s, min(s + step, E), dtype=torch.int64, device=dev)
        ci[s:s + step] = (e % N).to(torch.int32)
        ids[s:s + step] = e.to(torch.int32)
    vals = torch.empty(E, device=dev)

    def check_values(mode, what):
        say(what)
        for s in range(0, E, step):
            e = torch.arange(s, min(s + step, E), dtype=torch.int64, device=dev)
            deg = torch.where(e // d == M - 1, E - d * (M - 1), d).to(torch.float64)
            if mode == P.DR_NORM_MEAN:
                want = 1.0 / deg
            else:
                want = 1.0 / torch.sqrt(deg * (E // N + (e % N < E % N).to(torch.int64)).to(torch.float64))
            assert torch.equal(vals[s:s + step], want.to(torch.float32)), (what, s)

    for mode in (P.DR_NORM_MEAN, P.DR_NORM_SYM):
        ws = torch.empty(max(256, P.dr_csr_normalize_workspace_bytes(mode, M, N, E)), dtype=torch.uint8, device=dev)
        vals.zero_()
        P.dr_csr_normalize(mode, M, N, rp, ci, vals, ws)
        check_values(mode, f"normalize {mode}")
        del ws
        vals.zero_()
        P.dr_csr_normalize_noalloc(mode, M, N, rp, ci, vals)
        check_values(mode, f"normalize_noalloc {mode}")
    del vals
    say("transpose")
    At = P.device_transpose(P.Csr(M, N, rp, ci, ids.view(torch.float32)))
    c = torch.arange(N + 1, dtype=torch.int64, device=dev)
    start = c * (E // N) + torch.clamp(c, max=E % N)                      # the first E % N columns hold one entry more
    assert torch.equal(At.rowptr.to(torch.int64), start)
    got = At.vals.view(torch.int32)
    for s in range(0, E, step):
        at = torch.arange(s, min(s + step, E), dtype=torch.int64, device=dev)
        col = torch.searchsorted(start, at, right=True) - 1
        e = col + (at - start[col]) * N
        assert torch.equal(got[s:s + step].to(torch.int64), e), s
        assert torch.equal(At.colidx[s:s + step].to(torch.int64), e // d), s


@pytest.mark.parametrize("M,N,E,law", [
    # one bucket of 64 columns at the size up to which it is sorted in LDS
    (900, 64, 5119, "uniform"), (900, 64, 5120, "uniform"), (900, 64, 5121, "skewed_cols"),
    # tiles of two chunks, the second partly filled; rows that end far apart between them
    (300_000, 200_000, 4_300_000, "uniform"), (2_000_000, 200_000, 4_200_001, "tail_rows"),
])
def test_transpose_where_sorting_in_lds_changes(M, N, E, law):
    test_transpose_and_values_exact(M, N, E, law)


@pytest.mark.parametrize("M,N,E,law", [
    # two entries a column and one more: every second wavefront of the second level has counters, then every one
    (300_000, 1_100_000, 2_200_000, "uniform"), (300_000, 1_100_000, 2_200_001, "uniform"),
    (300_000, 5_000_000, 1_000_000, "skewed_cols"),
])
def test_transpose_of_wide_relations(M, N, E, law):
    test_transpose_and_values_exact(M, N, E, law)
