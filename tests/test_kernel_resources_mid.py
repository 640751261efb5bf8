"""The DR-SpMM kernels of 16 rows per wavefront keep nothing in scratch memory and leave room for as many wavefronts as those of 8
and 32 (checked on the compiler's own resource report, no GPU needed)."""
import re

from paper_2508_16769_amd import build


def test_kernels_of_sixteen_rows():
    rep = build.kernel_resources("spmm.hip")
    mid = {n: r for n, r in rep.items() if "spmm_fwd_mid_kernel" in n or "spmm_bwd_mid_kernel" in n or
           re.search(r"spmm_bwd_kernelILi\d+ELi\d+ELi16E", n)}
    assert len(mid) == 10 + 4 + 8, sorted(mid)            # forward by pairs per lane; backward: dense, compact uniform and adaptive
    for name, r in mid.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        if "ILi4ELi2E" in name:
            assert r["Occupancy"] >= 5, (name, r)
