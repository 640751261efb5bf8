// How the column partition of the per-graph setup (csr_ops.hip) splits a relation's entries between workgroups and
// wavefronts.  Plain C++, so that the ranges can be checked on the host at sizes no test can hold.
//
// Entry numbers are 32-bit and go up to 2^31 - 1, so the end of a range is never formed as begin + length before the
// length has been cut to what is there: begin + length may lie past 2^31.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define DRC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DRC_HOST_DEVICE inline
#endif

namespace drc {

constexpr int kPartThreads = 1024, kPartWaves = kPartThreads / 64;
constexpr int kMaxBuckets = 1024;      // level-1 digits: their counters (16 bits), one set per wavefront, take 32 KB of LDS
constexpr int kMaxSub = 2048;          // columns a workgroup of the second level owns: 128 KB of LDS counters, one set per wavefront
constexpr int kMinTile = 4096;         // entries a workgroup of the first level takes at least (256 per wavefront)
constexpr int kChunk = kMinTile;       // entries a workgroup of the first level sorts at a time, in LDS
constexpr int kMaxTiles = 1024;        // a chunk each up to 4.2 M entries; more would only lengthen the scan of the counts

struct PartShape {
    int shift;          // bucket = column >> shift
    int nb, nb_pad;     // buckets; rounded up to 64
    int sub_shift;      // columns a second-level workgroup owns = 1 << sub_shift (a bucket wider than kMaxSub is read by several)
    int tile, n_tiles;  // entries per first-level workgroup
};

inline PartShape part_shape(int64_t n_cols, int64_t nnz) {
    PartShape p;
    // Buckets of about 2048 entries (a second-level workgroup has two 64-entry steps per wavefront), at least 64 columns
    // wide and at most kMaxBuckets of them.
    p.shift = 6;
    while (((n_cols + (int64_t(1) << p.shift) - 1) >> p.shift) > kMaxBuckets) ++p.shift;
    while (p.shift < 11 && (nnz << p.shift) < 2048 * n_cols) ++p.shift;
    p.nb = (int)((n_cols + (int64_t(1) << p.shift) - 1) >> p.shift);
    if (p.nb < 1) p.nb = 1;
    p.nb_pad = (p.nb + 63) / 64 * 64;
    p.sub_shift = p.shift < 11 ? p.shift : 11;
    int64_t tile = (nnz + kMaxTiles - 1) / kMaxTiles;
    if (tile < kMinTile) tile = kMinTile;
    tile = (tile + kPartThreads - 1) / kPartThreads * kPartThreads;
    p.tile = (int)tile;
    p.n_tiles = (int)((nnz + tile - 1) / tile);
    return p;
}

struct PartRange { int begin, len; };      // entries [begin, begin + len)

// part `i` of a range cut into pieces of `per` (the last ones may be short or empty)
DRC_HOST_DEVICE PartRange part_piece(PartRange r, int i, int per) {
    const int64_t at = (int64_t)i * per;
    const int off = at < r.len ? (int)at : r.len;
    return PartRange{r.begin + off, r.len - off < per ? r.len - off : per};
}

// first level: the entries of workgroup `tile`, and of one of its wavefronts
DRC_HOST_DEVICE PartRange part_tile(const PartShape& p, int nnz, int tile) { return part_piece(PartRange{0, nnz}, tile, p.tile); }
DRC_HOST_DEVICE PartRange part_tile_wave(const PartShape& p, int nnz, int tile, int wave) {
    return part_piece(part_tile(p, nnz, tile), wave, p.tile / kPartWaves);
}

// second level: the stretch of a bucket of n records that one of the `waves` wavefronts takes (empty from there on)
DRC_HOST_DEVICE PartRange part_bucket_wave(int n, int wave, int waves = kPartWaves) {
    const int per = ((n - 1) / waves + 64) / 64 * 64;          // n / waves rounded up, then up to a multiple of 64
    return part_piece(PartRange{0, n}, wave, per);
}

}  // namespace drc
