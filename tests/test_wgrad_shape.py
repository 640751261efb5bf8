"""How many workgroups sum the rows of a weight gradient.  A running sum is in 32 bits and loses exactness with every row that is
added, so a graph of which one side fills the chip by itself must not give its sides fewer workgroups for sharing a launch.  The header
that defines the shares is plain C++ and is compiled here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "wgrad_shape.h"
#include <cstdio>
#include <initializer_list>
using namespace drc;
int main() {
    const int64_t full = int64_t(1) << 26;
    const struct { int D, chunk; } widths[] = {{32, 128}, {64, 64}, {96, 32}, {128, 32}};
    for (auto w : widths) {
        const int64_t edge = full / w.D;
        const int64_t rows[] = {0, 1, 31, 4097, 60000, edge - 1, edge, edge + 1, 2 * edge, 4 * edge};
        for (int64_t cells : rows)
            for (int64_t nets : rows)
                for (int res : {1, 104, 256, 512}) {
                    const WgradSide s[2] = {{cells, 3}, {nets, 2}};
                    int got[2];
                    for (int i = 0; i < 2; ++i) {
                        got[i] = wgrad_share(s, 2, i, w.D, w.chunk, res, full);
                        const int64_t most = wgrad_most((s[i].rows + w.chunk - 1) / w.chunk);        // what the scratch holds
                        if (got[i] < 1 || got[i] > most || (got[i] > res && got[i] > 1)) return printf("share %d\n", got[i]), 1;
                        const int alone = wgrad_share(s + i, 1, 0, w.D, w.chunk, res, full);
                        if ((cells > nets ? cells : nets) * w.D >= full && got[i] != alone)
                            return printf("D=%d %lld cells %lld nets: %d of %d\n", w.D, (long long)cells, (long long)nets, got[i], alone), 1;
                    }
                    if (cells * w.D < full && nets * w.D < full && got[0] + got[1] > (res < 256 ? res : 256) + 1) return puts("sum"), 1;
                }
    }
    puts("ok");
    return 0;
}
"""


def test_shares_of_weight_gradients(tmp_path):
    compiler = shutil.which("g++") or shutil.which("clang++")
    if compiler is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM)
    subprocess.run([compiler, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2508_16769_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
