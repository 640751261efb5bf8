// Rows that a wavefront of a DR-SpMM launch takes (spmm.hip).  Plain C++, so that the lines can be checked on the host.
#pragma once

#include <cstdint>

namespace drc {

constexpr int64_t kSmallLaunch = 8 * 24 * 256;   // rows of a launch with nets up to which a wavefront takes 8 of them

// Rows per wavefront.  More of them fill the groups evenly (a group that finishes takes the next row) and are planned at the cost of
// fewer; fewer of them put more wavefronts on the chip and cut the serial chain of a wavefront (8: one row per group).
//  * 8 while all wavefronts of a launch are resident at once, 256 compute units x 20 wavefronts; to 49 152 rows where a relation has fewer
//    rows than columns: nets, whose high-fanout rows are a workgroup's one after the other.  8 / 16 rows, us: 33 000 rows, D = 128,
//    k = 16, 10 edges per row forward 17.2 / 18.0, backward 17.6 / 18.4; 45 000 rows, k = 32 27.0 / 21.8 and 29.9 / 27.0; 42 000
//    nets, 42 of them with 200 to 2000 edges, 33 / 45 and 49 / 71.  (8 / 32 rows at 40 000 rows of 20 to 60 edges 51 / 101 and 105 / 114.)
//  * 32 above 2^19 rows of a relation, where the chip is full anyway (16 / 32: near of 1.2 M cells forward 436 / 412, with 8 edges per row
//    238 / 222; the layer's relations together, D = 64, forward 1 308 / 1 283, backward with dense rows 1 536 / 1 518).
//  * 16 in between, unless a wavefront's plan weighs too much.  What it weighs shows in the edges per row, what it brings in the number of
//    wavefronts; the lines lie where measured, 16 / 32 rows, us:
//    Forward, a relation alone.  Ten edges and more: 60 000 rows 26 / 34, 250 000, D = 128, k = 8 65 / 73, 500 000, k = 64 205 / 223.  (Power law
//    degrees at D = 64 and less lose up to a tenth past 300 000 rows: 350 000, k = 16 109 / 101.)  Less than nine: 80 000 rows 26 / 25,
//    120 000 31 / 25, 250 000, D = 64 45 / 39, so 32 as soon as wavefronts of 16 are not resident at once.  Nets differ most among their rows
//    and gain again when wavefronts of 32 are not resident either: 5 edges 84 000 nets 29 / 25, 112 000 35 / 32, 175 000 50 / 52,
//    280 000 77 / 78; 6.6 edges, hubs among them, 86 000 41 / 41, 144 000 53 / 62, 288 000 100 / 101.  Rows wider than 128 have larger row
//    buffers and fewer wavefronts resident: 60 000 rows of 3.5 edges, k = 32 D = 256 26 / 21, D = 512, k = 48 61 / 54; of 8 edges, D = 256 23 / 20.
//    Forward, relations sharing a launch (whole passes).  Up to 163 840 rows 16 gain at any degree: training steps of two sub-graphs 590 /
//    601, layers of 60 000 cells 125 / 128 to 355 / 363.  Up to 409 600 from six edges per row on: training on six sub-graphs of 6.3 edges
//    1 320 / 1 338, of 5.6 edges 1 189 / 1 172; layers of 130 000 cells 538 / 551 (from nine on without nets, as in a model's last layer: the
//    launch of eight sub-graphs, 320 000 rows of 6.8 edges, 82 / 80).  Above that from seven and a half on: training on eight
//    sub-graphs of 6.3 edges 1 603 / 1 585, layers of 300 000 cells of 7.6 1 220 / 1 234, of 7.0 527 / 516 (D = 32, 64) and 1 078 / 1 074.
//    Backward with dense rows: D = 32 layers of 130 000 / 180 000 / 250 000 / 450 000 cells 259 / 265, 340 / 333, 348 / 342, 753 / 729; D = 64
//    250 000 / 450 000 552 / 549, 1 129 / 1 111, training on eight sub-graphs 858 / 867; D = 128 up to 2^19 rows as fast or faster (1 087 / 1 094).
//    Backward, compact: at any size (1.2 M 530 / 580 near, 424 / 430 pins, 586 / 604 pinned, D = 128, k = 32) but for rows of D = 32 and less
//    than six edges: 130 000 rows, k = 16 24 / 21, 350 000 46 / 42, 1.2 M, k = 8 103 / 94 (90 000 18 / 20).
// The adaptive forward keeps 8 and 32 (16 at 250 000 rows: near 91 / 97, pins 86 / 82, pinned 64 / 61).
// Where 8 do not pay: a forward at D >= 256 or k = 128 with a few edges per row (D = 256, k = 32: 25 / 20 with 32, but 81 / 110 with 20 to
// 60 edges; there is a row buffer per group to clear, whatever the row brings).
struct LaunchShape {
    int64_t rows = 0, most = 0, nnz = 0;
    int relations = 0;
    bool nets = false;
    void add(int64_t n_rows, int64_t n_cols, int64_t n) {
        rows += n_rows;
        most = n_rows > most ? n_rows : most;
        nnz += n;
        ++relations;
        nets = nets || n_rows < n_cols;
    }
    // rows of as many wavefronts as fit 256 compute units at once: 20 each by their registers, fewer where four wavefronts' row buffers
    // of 8 x (D + 4) words and plans take more than a fifth of 160 KB
    static constexpr int64_t resident(int rows_per_wave, int D = 128) {
        const int groups = (160 << 10) / (16 * (8 * (D + 4) + 564));
        return (int64_t)rows_per_wave * 4 * (groups < 5 ? (groups < 1 ? 1 : groups) : 5) * 256;
    }
    bool eight() const { return rows <= (nets ? kSmallLaunch : resident(8)); }
    int forward(int D) const {
        if (eight()) return 8;
        if (most > int64_t(1) << 19) return 32;
        const bool few = nnz < (nets ? 6 : 9) * rows;
        if (relations > 1) return rows <= resident(32, D) || (!few && (rows <= resident(80, D) || 2 * nnz >= 15 * rows)) ? 16 : 32;
        return !few || rows <= resident(16, D) || (nets && rows > resident(32, D)) ? 16 : 32;
    }
    int forward_adaptive() const { return rows <= kSmallLaunch ? 8 : 32; }
    int compact(int D) const { return eight() ? 8 : D <= 32 && nnz < 6 * rows && rows > resident(20) ? 32 : 16; }
    int dense(int D) const { return eight() ? 8 : most <= int64_t(1) << 19 && rows <= 8192ll * D ? 16 : 32; }
};

}  // namespace drc
