"""The ranges into which the column partition of the per-graph setup cuts a relation's entries cover every entry once, up to
the largest accepted number of entries (2^31 - 1).  The header that defines them is plain C++ and is compiled here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "partition_shape.h"
#include <cstdio>
using namespace drc;
static long long g_at;
static bool next(PartRange r) {                 // consecutive, in bounds, no gap and no overlap
    if (r.len < 0 || (r.len > 0 && r.begin != g_at)) return false;
    g_at += r.len;
    return true;
}
int main() {
    const long long top = 1ll << 31;
    const long long sizes[] = {1, 63, 64, 4095, 4096, 4097, 2097151, 2097153, top - 262145, top - 262144, top - 262143, top - 262142,
                               top - 4097, top - 2049, top - 2048, top - 2047, top - 513, top - 256, top - 255, top - 65, top - 8, top - 7, top - 2, top - 1};
    const long long cols[] = {1, 64, 65536, 1300000, top - 3};
    for (long long n_cols : cols)
        for (long long n : sizes) {
            const PartShape p = part_shape(n_cols, n);
            if (p.nb < 1 || p.nb > kMaxBuckets || p.n_tiles < 1 || p.n_tiles > kMaxTiles) return printf("shape %lld %lld\n", n_cols, n), 1;
            g_at = 0;
            for (int t = 0; t < p.n_tiles; ++t)
                if (!next(part_tile(p, (int)n, t))) return printf("tile %d of %lld entries\n", t, n), 1;
            if (g_at != n) return printf("tiles cover %lld of %lld entries\n", g_at, n), 1;
            g_at = 0;
            for (int t = 0; t < p.n_tiles; ++t) {
                const PartRange r = part_tile(p, (int)n, t);
                for (int w = 0; w < kPartWaves; ++w)
                    if (!next(part_tile_wave(p, (int)n, t, w))) return printf("wavefront %d of tile %d of %lld entries\n", w, t, n), 1;
                if (g_at != (long long)r.begin + r.len) return printf("wavefronts of tile %d of %lld entries\n", t, n), 1;
            }
        }
    for (long long n : sizes) {                 // a bucket may hold everything
        g_at = 0;
        for (int w = 0; w < kPartWaves; ++w) {
            const PartRange r = part_bucket_wave((int)n, w);
            if (!next(r) || r.len > (1ll << 30)) return printf("wavefront %d of a bucket of %lld\n", w, n), 1;
        }
        if (g_at != n) return printf("wavefronts cover %lld of a bucket of %lld\n", g_at, n), 1;
    }
    for (long long n : sizes) {                 // fewer wavefronts take it: those past them get nothing
        g_at = 0;
        for (int w = 0; w < kPartWaves; ++w) {
            const PartRange r = part_bucket_wave((int)n, w, kPartWaves / 2);
            if (!next(r) || (w >= kPartWaves / 2 && r.len != 0)) return printf("wavefront %d of half of a bucket of %lld\n", w, n), 1;
        }
        if (g_at != n) return printf("half the wavefronts cover %lld of a bucket of %lld\n", g_at, n), 1;
    }
    puts("ok");
    return 0;
}
"""


def test_ranges_cover_every_entry_once(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "ranges.cpp", tmp_path / "ranges"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-fwrapv", "-I", os.path.join(ROOT, "paper_2508_16769_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
