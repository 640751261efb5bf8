"""What a launcher keeps per device is looked up once for each device, not once for the process, and a failed look-up is not
kept.  The header is plain C++ and is compiled here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "per_device.h"
#include <initializer_list>
#include <cstdio>
int main() {
    static drc::PerDevice kept;
    int looked[40] = {}, out = 0;
    auto ask = [&](int dev) { return kept.get(dev, &out, [&](int* n) { ++looked[dev]; *n = 100 + dev; return 0; }); };
    for (int round = 0; round < 3; ++round)
        for (int dev : {1, 0, 31, 33})
            if (ask(dev) != 0 || out != 100 + dev) return printf("device %d gave %d\n", dev, out), 1;
    if (looked[0] != 1 || looked[1] != 1 || looked[31] != 1 || looked[33] != 3) return puts("look-ups"), 1;
    if (kept.get(5, &out, [](int*) { return -3; }) != -3) return puts("a failure was not passed on"), 1;
    if (ask(5) != 0 || out != 105 || looked[5] != 1) return puts("a failure was kept"), 1;
    puts("ok");
    return 0;
}
"""


def test_kept_per_device(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "per_device.cpp", tmp_path / "per_device"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2508_16769_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
