"""How many rows a wavefront of a DR-SpMM launch takes: both sides of every line, and the launches that were slower with 16 rows than
with 32.  The header that defines the lines is plain C++ and is compiled here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "launch_shape.h"
#include <cstdio>
#include <initializer_list>
using namespace drc;
struct Rel { int64_t rows, cols, nnz; };
static LaunchShape shape(std::initializer_list<Rel> rels) {
    LaunchShape s;
    for (const Rel& r : rels) s.add(r.rows, r.cols, r.nnz);
    return s;
}
static int failures = 0;
#define EXPECT(value, want) if ((value) != (want)) ++failures, printf("line %d: %s is %d, not %d\n", __LINE__, #value, (int)(value), (int)(want))
static int alone(int64_t rows, int64_t cols, int64_t nnz, int D = 128) { return shape({{rows, cols, nnz}}).forward(D); }
// near, pins and pinned of a layer of so many cells and nets
static LaunchShape layer(int64_t cells, int64_t nets, int64_t near, int64_t pins) {
    return shape({{cells, cells, near}, {nets, cells, pins}, {cells, nets, pins}});
}
static LaunchShape dense(int64_t cells, int64_t nets) { return shape({{cells, cells, 0}, {nets, cells, 0}}); }
int main() {
    // 8 rows, with and without nets
    EXPECT(alone(40960, 3000, 0), 8);
    EXPECT(alone(40961, 3000, 0), 16);
    EXPECT(alone(49152, 50001, 0), 8);
    EXPECT(alone(49153, 50001, 0), 16);
    EXPECT(shape({{40961, 700, 0}}).compact(64), 16);
    EXPECT(dense(30000, 19152).dense(64), 8);
    EXPECT(dense(30000, 19153).dense(64), 16);
    // forward alone: edges per row, and 2^19 rows
    EXPECT(alone(81920, 900, 9 * 81920 - 1), 16);
    EXPECT(alone(81921, 900, 9 * 81921 - 1), 32);
    EXPECT(alone(81921, 900, 9 * 81921), 16);
    EXPECT(alone(81920, 900, 0, 32), 16);
    EXPECT(alone(81921, 900, 0, 32), 32);
    // wide rows, of which fewer are resident (60 000 rows of 3.5 edges, D = 256: 26 us with 16 rows, 21 with 32)
    EXPECT(alone(65536, 900, 0, 192), 16);
    EXPECT(alone(65537, 900, 0, 192), 32);
    EXPECT(alone(49152, 900, 0, 256), 16);
    EXPECT(alone(60000, 900, 210000, 256), 32);
    EXPECT(alone(60000, 900, 600000, 256), 16);
    EXPECT(alone(40961, 900, 0, 512), 32);
    EXPECT(alone(40961, 900, 0, 4096), 32);
    EXPECT(alone(524288, 70, 12 * 524288), 16);
    EXPECT(alone(524289, 70, 12 * 524289), 32);
    // nets: 112 000 of 5 edges took 35 us with 16 rows, 32 with 32
    EXPECT(alone(81920, 200000, 5 * 81920), 16);
    EXPECT(alone(112000, 160000, 5 * 112000), 32);
    EXPECT(alone(112000, 160000, 6 * 112000), 16);
    EXPECT(alone(163840, 200000, 5 * 163840), 32);
    EXPECT(alone(163841, 200000, 5 * 163841), 16);
    EXPECT(alone(524289, 900000, 5 * 524289), 32);
    // relations together: layers, and training on stacked sub-graphs of 20 000 cells (8: 1 603 us with 16 rows, 1 585 with 32)
    EXPECT(layer(60000, 40000, 480000, 200000).forward(128), 16);
    EXPECT(layer(81920, 81920, 0, 0).rows, 3 * 81920);
    EXPECT(shape({{81920, 81920, 0}, {81920, 81920, 0}}).forward(128), 16);
    EXPECT(shape({{81920, 81920, 0}, {81921, 81921, 0}}).forward(128), 32);
    EXPECT(layer(6 * 20000, 6 * 14000, 6 * 200000, 6 * 70000).forward(128), 16);
    EXPECT(layer(6 * 20000, 6 * 14000, 6 * 160000, 6 * 70000).forward(128), 32);
    EXPECT(layer(8 * 20000, 8 * 14000, 8 * 200000, 8 * 70000).forward(128), 32);
    EXPECT(layer(8 * 20000, 8 * 14000, 8 * 160000, 8 * 70000).forward(128), 32);
    EXPECT(layer(250000, 180000, 3000000, 1180000).forward(128), 16);
    // the last layer of a model: no nets
    EXPECT(shape({{46000, 46000, 460000}, {46000, 32000, 160000}}).forward(128), 16);
    EXPECT(shape({{160000, 160000, 1600000}, {160000, 112000, 560000}}).forward(128), 32);
    EXPECT(shape({{160000, 160000, 9 * 320000}, {160000, 112000, 0}}).forward(128), 16);
    EXPECT(layer(524288, 100000, 12 * 524288, 1500000).forward(128), 16);
    EXPECT(layer(524289, 100000, 12 * 524289, 1500000).forward(128), 32);
    // dense backward: narrow rows (250 000 cells, D = 32: 348 us with 16 rows, 342 with 32) and 2^19 rows
    EXPECT(dense(200000, 62144).dense(32), 16);
    EXPECT(dense(200000, 62145).dense(32), 32);
    EXPECT(dense(300000, 224288).dense(64), 16);
    EXPECT(dense(300000, 224289).dense(64), 32);
    EXPECT(dense(524288, 200000).dense(128), 16);
    EXPECT(dense(524289, 200000).dense(128), 32);
    // compact backward: narrow rows of few edges (350 000 x 3, D = 32, k = 16: 46 us with 16 rows, 42 with 32)
    EXPECT(shape({{102400, 70000, 300000}}).compact(32), 16);
    EXPECT(shape({{102401, 70000, 300000}}).compact(32), 32);
    EXPECT(shape({{102401, 70000, 6 * 102401}}).compact(32), 16);
    EXPECT(shape({{102401, 70000, 300000}}).compact(64), 16);
    EXPECT(shape({{49152, 1, 0}}).forward_adaptive(), 8);
    EXPECT(shape({{49153, 1, 0}}).forward_adaptive(), 32);
    if (!failures) puts("ok");
    return failures != 0;
}
"""


def test_rows_per_wavefront(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2508_16769_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
