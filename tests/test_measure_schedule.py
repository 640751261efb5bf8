"""Counter runs are attributed to the layer's kernels by dispatch order and by a part of the kernel's name: every kernel of the
layer's steps has to be found by it, whichever variant a size takes."""
import csv
import glob
import os
import re

import pytest

import measure

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernels():
    text = "".join(open(p).read() for p in glob.glob(os.path.join(ROOT, "paper_2508_16769_amd", "csrc", "*.hip")))
    return set(re.findall(r"__global__\s+(?:__launch_bounds__\([^;{]*?\)\s+)?void\s+(\w+)\s*\(", text))


def _rows(names, steps):
    return [dict(Dispatch_Id=str(i + 1), Kernel_Name=f"void drc::{n}<8, 4, false>(drc::Args)", Counter_Value=str(i % len(names)))
            for i, n in enumerate(list(names) * steps)]


@pytest.mark.parametrize("topk", ["topk_rows_kernel", "topk_groups_kernel"])
@pytest.mark.parametrize("schedule", [measure.SCHEDULE, measure.SCHEDULE_DR])
def test_counters_of_every_variant_are_attributed(tmp_path, topk, schedule):
    kernels = _kernels()
    assert topk in kernels
    names = []
    for label, part in schedule:
        hits = [k for k in kernels if part in k]
        assert hits, (label, part)
        names.append(topk if label.startswith("dr_topk") else sorted(hits)[0])
    path = tmp_path / "counters.csv"
    with open(path, "w", newline="") as fh:
        w = csv.DictWriter(fh, ["Dispatch_Id", "Kernel_Name", "Counter_Value"])
        w.writeheader()
        w.writerows(_rows(names, 3))
    got = measure.per_kernel_kib(str(path), schedule)
    assert got == {label: float(i) for i, (label, _) in enumerate(schedule)}
