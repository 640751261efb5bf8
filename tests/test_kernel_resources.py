"""The hot kernels keep nothing in scratch memory (checked on the compiler's own resource report, no GPU needed).

A scratch access is a vector-memory operation: the wavefront's wait for it also waits for every gather issued before
it, which once serialized the ping-pong batches of the DR-SpMM kernels (their per-group record stream had been placed
in scratch because one of its members was written on one side of a branch only).  The dense kernels at D = 128 fill the
256 registers of two wavefronts per SIMD almost to the last; their pipelines count the operations that may be outstanding, which
a spill would upset."""
import re
from concurrent.futures import ThreadPoolExecutor

from paper_2508_16769_amd import build


def _report():
    with ThreadPoolExecutor(max_workers=4) as pool:
        parts = list(pool.map(build.kernel_resources, ("topk.hip", "spmm.hip", "staged.hip", "dense.hip")))
    out = {}
    for p in parts:
        out.update(p)
    return out


def test_hot_kernels_use_no_scratch_memory():
    rep = _report()
    topk = {k: v for k, v in rep.items() if "topk_rows_kernel" in k or "topk_groups_kernel" in k}
    spmm = {k: v for k, v in rep.items() if "spmm_fwd_kernel" in k or "spmm_bwd_kernel" in k}
    staged = {k: v for k, v in rep.items() if "spmm_bwd_staged_kernel" in k}
    assert len(topk) >= 22 and len(spmm) >= 20 and len(staged) >= 16
    for name, r in {**topk, **spmm}.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (name, r)
    # staged tiles: the instantiations with 64-column slabs and up to 4 compact outputs per lane (k <= 64) hold their two
    # prefetch sets in registers; the widest ones (8 outputs per lane, k up to 128) are allowed to spill
    for name, r in staged.items():
        m = re.search(r"staged_kernelILi(\d+)ELi(\d+)ELi(\d+)E", name)
        cw, ks = int(m.group(1)), int(m.group(2))
        if cw == 64 and ks <= 4:
            assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (name, r)
    # the forward and backward kernels of the benchmark's width (k = 32) leave room for five wavefronts per SIMD or more:
    # pairs per lane, batch depth, rows per wavefront (8 or 32), not adaptive; the backward compact or dense
    k32 = {n: r for n, r in spmm.items() if re.search(r"spmm_(fwd|bwd)_kernelILi4ELi2ELi\d+ELb0E", n)}
    assert len(k32) == 6, sorted(k32)
    for name, r in k32.items():
        assert r["Occupancy"] >= 5, (name, r)
    dense = {n: r for n, r in rep.items() if re.search(r"\d(proj|dproj|wgrad_partial|wgrad_reduce|dense_bwd)_kernelILi", n)}
    assert len(dense) == 24, sorted(dense)           # four widths; the forward with two cache policies of its stores
    for name, r in dense.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0 and r["Occupancy"] >= 2, (name, r)
