// How the weight gradients of a backward pass are split between workgroups (dense.hip).  Plain C++, so that the shares can be
// checked on the host.
#pragma once

#include <cstdint>

namespace drc {

constexpr int kWgradMaxWgs = 256;                       // one workgroup per compute unit (its tiles take 147 KB of LDS)

// Most workgroups for a side (one node type of one graph) of so many chunks of rows.
// At least two chunks per workgroup: the partial sums a workgroup writes weigh as much as the rows of four chunks.  Up to
// kWgradSingle of them a chunk each all the same: half the chip is idle then, and a second chunk only lengthens the launch
// (whole layers, two / one chunk: 2048 cells, D = 64 69.8 / 67.8 us; 3000, 128 95.4 / 94.0; 8000, 64 and 128 the same).
constexpr int kWgradSingle = 128;
inline int64_t wgrad_most(int64_t chunks) {
    const int64_t single = chunks < kWgradSingle ? chunks : kWgradSingle, half = (chunks + 1) / 2;
    const int64_t n = half > single ? half : single;
    return n > kWgradMaxWgs ? kWgradMaxWgs : (n < 1 ? 1 : n);
}

struct WgradSide { int64_t rows; int products; };

// Workgroups of side i of n (cells and nets of a graph in turn, or one side alone); `res` of them fill the chip.  The sides of a launch
// share the chip by their work.  A graph of which one side fills the chip by itself (`full` elements) gets `res` for either side, as if
// they had a launch each: a workgroup's running sums are in 32 bits, and their error grows with the rows that it walks.  (1.2 M cells
// and 0.9 M nets, D = 128, N(0,1) data, shared / `res` for either: errors 2.7e-7 and 3.3e-7 / 2.2e-7 and 2.0e-7; the backward pass takes
// as long, 2 470 / 2 469 us.)
inline int wgrad_share(const WgradSide* s, int n, int i, int D, int chunk_rows, int res, int64_t full) {
    if (res > kWgradMaxWgs) res = kWgradMaxWgs;
    int64_t work = 0;
    for (int j = 0; j < n; ++j) work += s[j].rows * s[j].products;
    const int other = i ^ 1;
    const int64_t larger = other < n && s[other].rows > s[i].rows ? s[other].rows : s[i].rows;
    const int64_t wanted = larger * D >= full ? res : (work ? s[i].rows * s[i].products * res / work : 1);
    const int64_t most = wgrad_most((s[i].rows + chunk_rows - 1) / chunk_rows);
    return (int)(wanted < 1 ? 1 : (wanted > most ? most : wanted));
}

}  // namespace drc
