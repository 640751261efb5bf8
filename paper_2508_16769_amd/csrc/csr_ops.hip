// Per-graph setup kernels: module edge values (mean / symmetric normalisation) and the stable CSR
// transpose used by the backward pass (paper Alg. 2, stage 1).
#include "dr_internal.h"

#include <type_traits>
#include "partition_shape.h"

#include <mutex>

namespace drc {

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

int launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
    if (n == 0) return DR_OK;
    size_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

// ---------------------------------------------------------------------------------------------------
// Row of an edge.  A wavefront walks consecutive edges, 64 at a time.  The row of its first edge comes from a search
// that narrows 64-fold per load (four dependent loads for a million rows; a binary search per edge took twenty and was
// what bound these kernels); from there on every step loads the next 64 row ends once and each lane counts, through
// lane shuffles, how many of them lie at or before its own edge.  A run of empty rows between two edges is walked for
// kScanWindows windows and then jumped by another search: the loads of a step stay bounded whatever the rows look like (a
// gap of a million empty rows took 6.4 ms to walk, 64 rows per 0.4 us).
// ---------------------------------------------------------------------------------------------------
constexpr int kScanWindows = 4;       // as many dependent loads as a search in a million rows

// largest row with rowptr[row] <= e (rows may be empty), given a row `lo` with rowptr[lo] <= e; both are the same in every
// lane, 0 <= e < rowptr[n_rows]
__device__ __forceinline__ int wave_row_of(const int32_t* __restrict__ rowptr, int n_rows, int lo, int e) {
    const int lane = threadIdx.x & 63;
    int hi = n_rows;                                           // rowptr[lo] <= e < rowptr[hi]
    while (hi - lo > 1) {
        const int step = (int)(((unsigned)(hi - lo) + 63u) / 64u);
        const long long p = (long long)lo + (long long)step * (lane + 1);
        const bool below = p < hi && rowptr[p < hi ? (int)p : lo] <= e;
        const int n = __popcll(__ballot(below));               // the probes are sorted: the lanes below are a prefix
        const long long top = (long long)lo + (long long)step * (n + 1);
        lo += step * n;
        hi = top < hi ? (int)top : hi;
    }
    return lo;
}

// the same for an edge that is likely to lie within the next 4096 rows: at most 64 rows before the edge's, after one load
__device__ __forceinline__ int wave_row_ahead(const int32_t* __restrict__ rowptr, int n_rows, int lo, int e) {
    const long long p = (long long)lo + 64ll * ((threadIdx.x & 63) + 1);
    const bool below = p < n_rows && rowptr[p < n_rows ? (int)p : lo] <= e;
    const int n = __popcll(__ballot(below));
    return n < 64 ? lo + 64 * n : wave_row_of(rowptr, n_rows, lo + 64 * 64, e);
}

// The row ends a wavefront has at hand, kept from one step to the next: lane l holds the end of row base + l, and of the row
// 64 further on.  64 row ends serve a dozen steps where rows have a dozen edges; loaded anew for every step they were a
// dependent load per step, which is what these kernels waited for.
struct RowWindow { int base, start, end, next; };      // start = rowptr[base]

__device__ __forceinline__ int row_end(const int32_t* __restrict__ rowptr, int n_rows, uint32_t row) {
    return row < (uint32_t)n_rows ? rowptr[row + 1u] : 0x7fffffff;             // row may lie past 2^31
}
__device__ __forceinline__ RowWindow row_window(const int32_t* __restrict__ rowptr, int n_rows, int base) {
    const uint32_t at = (uint32_t)base + (uint32_t)(threadIdx.x & 63);
    return RowWindow{base, rowptr[base], row_end(rowptr, n_rows, at), row_end(rowptr, n_rows, at + 64u)};
}

// row of this lane's edge e and that row's number of edges, given a window whose first row is at or before the row of the
// wavefront's first edge; e rises with the lane, and from call to call
__device__ __forceinline__ int wave_rows(const int32_t* __restrict__ rowptr, int n_rows, RowWindow& w, int e, int* len) {
    int row = w.base;
    bool open = true;
    for (int window = 1;; ++window) {
        int c = 0;                                             // row ends at or before e among these 64 (sorted)
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) c += (__shfl(w.end, c + d - 1, 64) <= e) ? d : 0;
        const int at_c = __shfl(w.end, c, 64), below = __shfl(w.end, max(c - 1, 0), 64);
        const bool past = at_c <= e;                           // c = 63 here: all 64
        if (open) {
            row = w.base + c;
            *len = at_c - (c == 0 ? w.start : below);
        }
        open = open && past;
        const unsigned long long still = __ballot(open);
        if (!still) return row;
        const int base = w.base + 64;                          // rowptr[base] <= e of every open lane
        if (window % kScanWindows == 0) {
            w = row_window(rowptr, n_rows, wave_row_of(rowptr, n_rows, base, __builtin_amdgcn_readlane(e, __ffsll((long long)still) - 1)));
        } else {
            w.start = __builtin_amdgcn_readlane(w.end, 63);
            w.end = w.next;
            w.base = base;
            w.next = row_end(rowptr, n_rows, (uint32_t)base + (uint32_t)(threadIdx.x & 63) + 64u);
        }
    }
}

// Column counts with atomics: the columns a workgroup sees first are counted in LDS (one slot per column modulo the table),
// the others straight in memory, so a column that holds very many entries does not queue them all up at one address (9 ns each).
constexpr int kCountSlots = 2048, kCountPer = 8;
__global__ __launch_bounds__(256) void count_columns_kernel(const int32_t* __restrict__ colidx, int nnz, int32_t* __restrict__ count) {
    __shared__ int32_t tag[kCountSlots], cnt[kCountSlots];
    for (int i = threadIdx.x; i < kCountSlots; i += 256) { tag[i] = -1; cnt[i] = 0; }
    const uint32_t at = blockIdx.x * (uint32_t)(256 * kCountPer);
    const int left = min(nnz - (int)at, 256 * kCountPer);
    int32_t c[kCountPer];
#pragma unroll
    for (int u = 0; u < kCountPer; ++u) c[u] = colidx[(int)at + min((int)threadIdx.x + 256 * u, left - 1)];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCountPer; ++u) {
        if ((int)threadIdx.x + 256 * u >= left) continue;
        const int slot = c[u] & (kCountSlots - 1);
        const int32_t was = atomicCAS(&tag[slot], -1, c[u]);
        if (was == -1 || was == c[u]) atomicAdd(&cnt[slot], 1);
        else atomicAdd(&count[c[u]], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCountSlots; i += 256)
        if (cnt[i]) atomicAdd(&count[tag[i]], cnt[i]);
}
static int launch_count_columns(const int32_t* colidx, int64_t n_cols, int64_t nnz, int32_t* count, hipStream_t s) {
    DRC_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(count), (size_t)n_cols, 0u, s));
    hipLaunchKernelGGL(count_columns_kernel, dim3((unsigned)((nnz + 256 * kCountPer - 1) / (256 * kCountPer))), dim3(256), 0, s, colidx,
                       (int)nnz, count);
    return DR_OK;
}

// Edge values.  A wavefront takes `steps` * 64 consecutive edges, one step after the other: eight steps pay for the search of
// its first row, but while there are fewer steps in all than wavefronts that fill the chip, every step is a wavefront.
constexpr int kNormSteps = 8;
constexpr int kNormBatch = 4;         // steps whose column counts are requested together
__global__ __launch_bounds__(256) void normalize_kernel(int mode, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                        int n_rows, int nnz, const int32_t* __restrict__ deg_out,
                                                        float* __restrict__ vals, int steps) {
    const int lane = threadIdx.x & 63;
    const uint32_t at = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (uint32_t)(steps * 64);
    if (at >= (uint32_t)nnz) return;
    const int first = (int)at, left = min(nnz - first, steps * 64);
    RowWindow win = row_window(rowptr, n_rows, wave_row_of(rowptr, n_rows, 0, first));
    for (int s0 = 0; s0 < left; s0 += 64 * kNormBatch) {
        int dj[kNormBatch];
        if (mode != DR_NORM_MEAN) {
#pragma unroll
            for (int u = 0; u < kNormBatch; ++u) dj[u] = colidx[first + min(s0 + 64 * u + lane, left - 1)];
#pragma unroll
            for (int u = 0; u < kNormBatch; ++u) dj[u] = deg_out[dj[u]];
        }
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) {
            const int s = s0 + 64 * u;
            if (s >= left) break;
            const int e = first + min(s + lane, left - 1);
            int di;
            wave_rows(rowptr, n_rows, win, e, &di);
            float v;
            if (mode == DR_NORM_MEAN) {
                v = (float)(1.0 / (double)di);
            } else {
                const double a = (double)(di > 1 ? di : 1) * (double)(dj[u] > 1 ? dj[u] : 1);
                v = (float)(1.0 / sqrt(a));
            }
            if (s + lane < left) vals[e] = v;
        }
    }
}

static int launch_normalize_kernel(int mode, int64_t n_rows, int64_t nnz, const int32_t* rowptr, const int32_t* colidx,
                                   const int32_t* deg_out, float* vals_out, hipStream_t s) {
    int64_t steps = nnz / (64 * 4096);          // 256 compute units x 16 wavefronts
    steps = steps < 1 ? 1 : (steps > kNormSteps ? kNormSteps : steps);
    const unsigned blocks = (unsigned)((nnz + 4 * steps * 64 - 1) / (4 * steps * 64));
    hipLaunchKernelGGL(normalize_kernel, dim3(blocks), dim3(256), 0, s, mode, rowptr, colidx, (int)n_rows, (int)nnz, deg_out,
                       vals_out, (int)steps);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

// ---------------------------------------------------------------------------------------------------
// Edge values without a workspace argument: the column counts live in a device array that is part of the
// library image.  The array's name is only a host-side handle; its device address is looked up once per
// device and that pointer is what the kernels and the fill receive.
// ---------------------------------------------------------------------------------------------------

static __device__ __align__(256) int32_t scratch[DR_NOALLOC_MAX_COLS + 64];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static int32_t* g_scratch_ptr[kMaxDevices] = {};

static int scratch_of_current_device(int32_t** out) {
    int dev = -1;
    DRC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(DR_ERR_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        DRC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (p == nullptr) return fail(DR_ERR_HIP, "hipGetSymbolAddress returned a null address for the scratch array");
        g_scratch_ptr[dev] = static_cast<int32_t*>(p);
    }
    *out = g_scratch_ptr[dev];
    return DR_OK;
}

int launch_csr_normalize_noalloc(int mode, int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t* rowptr,
                                 const int32_t* colidx, float* vals_out, hipStream_t s) {
    int32_t* deg_out = nullptr;
    if (mode == DR_NORM_SYM) {       // no room for the column partition of the workspace variant: counted with atomics
        DRC_TRY(scratch_of_current_device(&deg_out));
        DRC_TRY(launch_count_columns(colidx, n_cols, nnz, deg_out, s));
    }
    return launch_normalize_kernel(mode, n_rows, nnz, rowptr, colidx, deg_out, vals_out, s);
}

// ---------------------------------------------------------------------------------------------------
// Stable transpose: a two-level stable counting sort of the entries by column.
//   1. part_count    a workgroup counts, in LDS, how many entries of its range of edges fall into each of at most 1024
//                    column buckets
//   2. part_scan     per bucket, the exclusive prefix of those counts over the workgroups, and the bucket's total
//   3. part_scatter  every entry moves to its bucket as a record (column, row, value), in storage order
//   4. part_columns  a workgroup sorts one bucket's records by column, in order, and writes its stretch of the transpose
//                    (and of the row pointers).  The symmetric edge values only need the column counts of this step.
// In steps 3 and 4 a wavefront takes a contiguous stretch of entries, 64 at a time; lanes with the same digit find each
// other with one ballot per digit bit, so an entry's place is the wavefront's running count of its digit (LDS) plus the
// number of lower lanes with the same digit: the order of equal digits is kept, and there are no atomics on memory.
// 44 bytes per entry move: column twice, value, record out and in, result.  Entries are put in order in LDS before they are
// written (steps 3 and 4): one by one, random columns made a memory transaction of every 4- or 8-byte store, and those bounded
// both steps.  Edge values and transposes of the three relations, before / after: 250 000 cells (3.0 / 1.2 / 1.2 M entries)
// 243 / 232 us (225 with the column counts in any order), 500 000 cells 431 / 334 (with all of this file's changes to step 2 and the
// row ends), 1.1 M cells 1455 / 1067 (mostly step 3: step 4 sorts in LDS where no relation of the batch has workgroups of 2048 columns).
// What bounds it now: 19 launches of 4 to 33 us one behind the other, each a chain of a dozen waits.
// (Earlier: one slot per entry by an atomic cursor and a ranking of every segment afterwards.  The random atomics, one binary
// search per entry and the ranking of the segments of high-fanout nets took 0.30 / 0.20 / 0.24 ms for the three relations of a
// 250 000-cell graph.)
// All three relations of a context go through one set of launches.
// ---------------------------------------------------------------------------------------------------

struct PartSeg {
    PartShape p;
    const int32_t *rowptr, *colidx;
    const float* vals;
    int n_rows, n_cols, nnz;
    int32_t *t_rowptr, *t_colidx;      // t_rowptr: row pointers of the transpose, or (count only) the column counts
    float* t_vals;
    uint32_t *hist, *totals;           // [n_tiles][nb_pad], [nb_pad]
    int32_t* key;                      // [nnz] columns in bucket order
    int2* rec;                         // [nnz] (row, value bits) in bucket order
    int count_only;
    int tile0, scan0, col0;            // first workgroup of this relation in the launches of steps 1 and 3 / 2 / 4
};
constexpr int kMaxPartSegs = 4;
constexpr int kPartBatch = 4;      // loads of entries a lane has in flight
struct PartBatch { PartSeg s[kMaxPartSegs]; int n; };

// inclusive scan of one value per thread of the workgroup; every thread gets its own prefix
__device__ __forceinline__ uint32_t part_scan_inclusive(uint32_t v, uint32_t* smem /* [kPartWaves] */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    __syncthreads();
    if (lane == 63) smem[wave] = x;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < kPartWaves; ++w) before += w < wave ? smem[w] : 0u;
    return x + before;
}

__global__ __launch_bounds__(kPartThreads) void part_count_kernel(PartBatch b) {
    __shared__ uint32_t cnt[kMaxBuckets];
    int q = 0;
    while (q + 1 < b.n && (int)blockIdx.x >= b.s[q + 1].tile0) ++q;
    const PartSeg& g = b.s[q];
    const int tile = blockIdx.x - g.tile0;
    const PartRange r = part_tile_wave(g.p, g.nnz, tile, threadIdx.x >> 6);     // may be empty in the last tile: begins past 0 then
    const int lane = threadIdx.x & 63;
    const int32_t* const col = g.colidx + r.begin;
    int c[kPartBatch];                                      // the first loads fly while the counters are cleared
#pragma unroll
    for (int u = 0; u < kPartBatch; ++u) c[u] = col[min(lane + u * 64, r.len - 1)];
    for (int i = threadIdx.x; i < g.p.nb_pad; i += kPartThreads) cnt[i] = 0u;
    __syncthreads();
    for (int i = lane; i < r.len; i += kPartBatch * 64) {
        int next[kPartBatch];
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u) next[u] = col[min(i + (kPartBatch + u) * 64, r.len - 1)];
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u) {
            if (i + u * 64 < r.len) atomicAdd(&cnt[c[u] >> g.p.shift], 1u);
            c[u] = next[u];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < g.p.nb_pad; i += kPartThreads) g.hist[(size_t)tile * g.p.nb_pad + i] = cnt[i];
}

// 64 buckets per workgroup (one per lane); the 16 wavefronts split the tiles.  There are only a handful of workgroups: the
// time is that of the chain of loads, so a wavefront requests all its counts at once and keeps them.
constexpr int kScanPer = kMaxTiles / 16;
__global__ __launch_bounds__(1024) void part_scan_kernel(PartBatch b) {
    __shared__ uint32_t sum[16][64];
    int q = 0;
    while (q + 1 < b.n && (int)blockIdx.x >= b.s[q + 1].scan0) ++q;
    const PartSeg& g = b.s[q];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_tiles = g.p.n_tiles, nb_pad = g.p.nb_pad, per = (n_tiles + 15) / 16;       // per <= kScanPer
    const int t0 = min(wave * per, n_tiles), n = min(per, n_tiles - t0);
    uint32_t* const h = g.hist + (blockIdx.x - g.scan0) * 64 + lane + (size_t)t0 * nb_pad;
    uint32_t v[kScanPer], s = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; j += 8) {
#pragma unroll
        for (int u = j; u < j + 8; ++u) v[u] = 0u;
        if (j < n) {
#pragma unroll
            for (int u = j; u < j + 8; ++u) v[u] = h[(size_t)min(u, n - 1) * nb_pad];
        }
    }
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) s += u < n ? v[u] : 0u;
    sum[wave][lane] = s;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        run += w < wave ? sum[w][lane] : 0u;
        total += sum[w][lane];
    }
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) {
        if (u < n) h[(size_t)u * nb_pad] = run;
        run += v[u];
    }
    if (wave == 0) g.totals[(blockIdx.x - g.scan0) * 64 + lane] = total;
}

// lanes of the wavefront with this lane's digit (bits [0, nbits)), among the lanes where `on` holds
__device__ __forceinline__ unsigned long long same_digit(uint32_t digit, int nbits, bool on) {
    unsigned long long m = __ballot(on);
    for (int i = 0; i < nbits; ++i) {
        const bool bit = (digit >> i) & 1u;
        const unsigned long long v = __ballot(bit);
        m &= bit ? v : ~v;
    }
    return m;
}
__device__ __forceinline__ int bits_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A chunk of the tile is sorted by bucket in LDS and leaves in that order, so that neighbouring lanes write neighbouring records:
// written straight from the entries' order every lane's record was a transaction of its own, and those were what the kernel
// took (1.2 M entries into 489 buckets 28 us, whether 8 or 16 wavefronts worked on a tile; without the records 13).
__host__ __device__ constexpr size_t scatter_lds(int nb_pad) { return 2 * (size_t)kPartWaves * nb_pad + 12 * (size_t)kChunk; }
using Count16 = uint16_t __attribute__((may_alias));
// RECORDS false: columns only, of which nothing but counts is made, so that any order will do within a bucket and places come from LDS
// atomics.  Ranked like records, columns that lie near their bucket already took longer than written one by one: symmetric edge
// values of 1.2 M x 0.9 M with 5 M entries near the diagonal 100 us without the sorting, 121 with it, 97 now; random columns 128,
// 119, 101.  (A kernel of its own: with both ways in one the registers of the other spilled, transposes 3 to 12 % slower.)
template <bool RECORDS>
__global__ __launch_bounds__(kPartThreads, 8) void part_scatter_kernel(PartBatch b) {
    static_assert(kMaxBuckets <= kPartThreads && kChunk % kPartThreads == 0 && kChunk < 65536, "one bucket per thread, 16-bit places");
    constexpr int kSteps = kChunk / kPartThreads;
    extern __shared__ __align__(16) uint32_t cnt[];                       // [kPartWaves][nb_pad] 16-bit counts, then places in the chunk
    int q = 0;
    while (q + 1 < b.n && (int)blockIdx.x >= b.s[q + 1].tile0) ++q;
    const PartSeg& g = b.s[q];
    const int tile = blockIdx.x - g.tile0, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, bucket = threadIdx.x;
    const int nbp = g.p.nb_pad, shift = g.p.shift, nbits = 32 - __builtin_clz(max(g.p.nb - 1, 1));
    const bool have = bucket < nbp;
    uint32_t* const s_key = cnt + kPartWaves * nbp / 2;      // [kChunk] columns, sorted
    int2* const s_rec = reinterpret_cast<int2*>(s_key + kChunk);
    uint32_t* const sm = s_key;                              // [kPartWaves] of the scans, which end before the sorting begins
    Count16* const place = reinterpret_cast<Count16*>(cnt);
    Count16* const mine = place + wave * nbp;
    // where this tile's next record of the thread's bucket goes: bucket start + what earlier tiles put there
    const uint32_t total = have ? g.totals[bucket] : 0u, prefix = have ? g.hist[(size_t)tile * nbp + bucket] : 0u;
    uint32_t next = part_scan_inclusive(total, sm) - total + prefix;
    const PartRange whole = part_tile(g.p, g.nnz, tile);
    int row0 = 0;
    for (int at_chunk = 0, k = 0; at_chunk < whole.len; at_chunk += kChunk, ++k) {
        const PartRange chunk = part_piece(whole, k, kChunk), r = part_piece(chunk, wave, kChunk / kPartWaves);
        if constexpr (!RECORDS) {
            int col[kSteps];
            uint32_t rank[kSteps];
#pragma unroll
            for (int u = 0; u < kSteps; ++u) col[u] = g.colidx[chunk.begin + min(u * kPartThreads + (int)threadIdx.x, chunk.len - 1)];
            if (have) cnt[bucket] = 0u;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kSteps; ++u)
                if (u * kPartThreads + (int)threadIdx.x < chunk.len) rank[u] = atomicAdd(&cnt[(uint32_t)col[u] >> shift], 1u);
            __syncthreads();
            const uint32_t n = have ? cnt[bucket] : 0u, local = part_scan_inclusive(n, sm) - n;
            if (have) cnt[bucket] = local;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kSteps; ++u)
                if (u * kPartThreads + (int)threadIdx.x < chunk.len) s_key[cnt[(uint32_t)col[u] >> shift] + rank[u]] = (uint32_t)col[u];
            __syncthreads();
            if (have) cnt[bucket] = next - local;
            next += n;
            __syncthreads();
            for (int i = threadIdx.x; i < chunk.len; i += kPartThreads) {
                const uint32_t key = s_key[i];
                g.key[cnt[key >> shift] + (uint32_t)i] = (int32_t)key;
            }
            __syncthreads();
            continue;
        }
        int c[kSteps];
        float v0 = 0.0f;
        RowWindow win{};
        for (int i = threadIdx.x; i < kPartWaves * nbp / 2; i += kPartThreads) cnt[i] = 0u;
        if (r.len > 0) {
#pragma unroll
            for (int u = 0; u < kSteps; ++u) c[u] = g.colidx[r.begin + min(u * 64 + lane, r.len - 1)];
            if constexpr (RECORDS) {
                if (g.vals) v0 = g.vals[r.begin + min(lane, r.len - 1)];
                row0 = k == 0 ? wave_row_of(g.rowptr, g.n_rows, 0, r.begin) : wave_row_ahead(g.rowptr, g.n_rows, row0, r.begin);
                win = row_window(g.rowptr, g.n_rows, row0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSteps; ++u)
            if (u * 64 + lane < r.len) {
                const uint32_t d = (uint32_t)c[u] >> shift;
                atomicAdd(&cnt[(wave * nbp + d) >> 1], 1u << (16 * (d & 1u)));       // nb_pad is even
            }
        __syncthreads();
        uint32_t n = 0;
        if (have)
#pragma unroll 4                                            // all sixteen at once take the registers past 64
            for (int w = 0; w < kPartWaves; ++w) n += place[w * nbp + bucket];
        const uint32_t local = part_scan_inclusive(n, sm) - n;
        if (have) {
            uint32_t at = local;
            for (int w = 0; w < kPartWaves; ++w) {
                const uint32_t m = place[w * nbp + bucket];
                place[w * nbp + bucket] = (uint16_t)at;
                at += m;
            }
        }
        __syncthreads();
        // The columns of the later steps are read again, one step ahead: kept from above they and their unrolled steps take 82
        // registers, and two workgroups no longer fit a compute unit.
        int col = c[0];
#pragma unroll 1
        for (int s = 0; s < r.len; s += 64) {
            const int e = r.begin + min(s + lane, r.len - 1), e_next = r.begin + min(s + 64 + lane, r.len - 1);
            const int col_next = g.colidx[e_next];
            const float v_next = RECORDS && g.vals ? g.vals[e_next] : 0.0f;
            const bool on = s + lane < r.len;
            const uint32_t d = (uint32_t)col >> shift;
            const unsigned long long m = same_digit(d, nbits, on);
            const uint32_t at = mine[d];
            const int before = bits_below(m);
            __builtin_amdgcn_wave_barrier();                // one wavefront's LDS accesses run in program order
            if (on && before == __popcll(m) - 1) mine[d] = (uint16_t)(at + (uint32_t)before + 1u);
            __builtin_amdgcn_wave_barrier();
            if constexpr (RECORDS) {
                int len;
                const int i = wave_rows(g.rowptr, g.n_rows, win, e, &len);
                if (on) s_rec[at + before] = make_int2(i, __float_as_int(v0));
            }
            if (on) s_key[at + before] = (uint32_t)col;
            col = col_next;
            v0 = v_next;
        }
        __syncthreads();
        if (have) cnt[bucket] = next - local;               // the places are used up: from place in the chunk to place in memory
        next += n;
        __syncthreads();
        for (int i = threadIdx.x; i < chunk.len; i += kPartThreads) {
            const uint32_t key = s_key[i], at = cnt[key >> shift] + (uint32_t)i;
            g.key[at] = (int32_t)key;
            if constexpr (RECORDS) g.rec[at] = s_rec[i];
        }
        __syncthreads();
    }
}

// Counters: a set for each wavefront, or (HALVE) for every second one where the workgroup owns kMaxSub columns; the other wavefronts
// then only clear and write.
template <bool HALVE>
__global__ __launch_bounds__(kPartThreads) void part_columns_kernel(PartBatch b, int sort_cap) {
    extern __shared__ __align__(16) uint32_t cnt[];                       // [sets][columns of this workgroup]; [sort_cap] records
    __shared__ uint32_t sm[kPartWaves];
    __shared__ uint32_t s_begin, s_before, s_total;
    int q = 0;
    while (q + 1 < b.n && (int)blockIdx.x >= b.s[q + 1].col0) ++q;
    const PartSeg& g = b.s[q];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = 1 << g.p.sub_shift, sets = HALVE && sub == kMaxSub ? kPartWaves / 2 : kPartWaves;
    const int first = (int)min((long long)(blockIdx.x - g.col0) << g.p.sub_shift, (long long)g.n_cols);    // first column
    const int ncol = min(sub, g.n_cols - first);
    const int bucket = first >> g.p.shift;
    if (ncol <= 0) return;
    for (int i = threadIdx.x; i < sets * sub; i += kPartThreads) cnt[i] = 0u;
    // records of the bucket: [begin, begin + n)
    uint32_t t = 0;
    for (int i = threadIdx.x; i < bucket; i += kPartThreads) t += g.totals[i];
    t = part_scan_inclusive(t, sm);
    if (threadIdx.x == kPartThreads - 1) s_begin = t;
    if (threadIdx.x == 0) s_before = 0u;
    __syncthreads();
    const int begin = (int)s_begin, n = (int)g.totals[bucket];
    const PartRange w = part_bucket_wave(n, wave, sets);      // wavefronts without counters: empty
    uint32_t* const mine = cnt + wave * sub;
    const int32_t* key = g.key + begin + w.begin;
    uint32_t earlier = 0;                                   // records of the bucket in columns before this workgroup's
    for (int i = lane; i < w.len; i += kPartBatch * 64) {
        int c[kPartBatch];
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u) c[u] = key[min(i + u * 64, w.len - 1)] - first;
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u)
            if (i + u * 64 < w.len) {
                if (c[u] >= 0 && c[u] < ncol) atomicAdd(&mine[c[u]], 1u);
                earlier += c[u] < 0 ? 1u : 0u;
            }
    }
    if (earlier) atomicAdd(&s_before, earlier);
    __syncthreads();
    // column starts: kPer consecutive columns per thread; the counters become next free places.  False: only counts were asked for.
    const auto column_starts = [&](auto n_sets) {
        constexpr int kSets = decltype(n_sets)::value, kPer = kMaxSub / kPartThreads;
        uint32_t col[kPer], sum = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = threadIdx.x * kPer + u;
            col[u] = 0u;
            if (i < sub)
                for (int w = 0; w < kSets; ++w) col[u] += cnt[w * sub + i];
            sum += col[u];
        }
        if (g.count_only) {
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int i = threadIdx.x * kPer + u;
                if (i < ncol) g.t_rowptr[first + i] = (int32_t)col[u];
            }
            return false;
        }
        const uint32_t incl = part_scan_inclusive(sum, sm);
        if (threadIdx.x == kPartThreads - 1) s_total = incl;
        uint32_t run = (uint32_t)begin + s_before + incl - sum;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = threadIdx.x * kPer + u;
            if (i < ncol) {
                g.t_rowptr[first + i] = (int32_t)run;
                uint32_t at = run;
                for (int w = 0; w < kSets; ++w) {
                    const uint32_t k = cnt[w * sub + i];
                    cnt[w * sub + i] = at;
                    at += k;
                }
            }
            run += col[u];
        }
        return true;
    };
    if (!(sets == kPartWaves ? column_starts(std::integral_constant<int, kPartWaves>{})
                             : column_starts(std::integral_constant<int, kPartWaves / 2>{}))) return;
    if (first + ncol == g.n_cols && threadIdx.x == 0) g.t_rowptr[g.n_cols] = g.nnz;
    __syncthreads();
    // A bucket that fits is sorted in LDS and leaves in order, coalesced; a larger one, and all of them where the batch's counters leave
    // no room (sort_cap = 0), is written record by record.
    int2* const s_out = reinterpret_cast<int2*>(cnt + sets * sub);
    const bool sorted = n <= sort_cap;
    const uint32_t origin = (uint32_t)begin + s_before;     // first place of this workgroup's columns
    const int2* rec = g.rec + begin + w.begin;
    for (int s0 = 0; s0 < w.len; s0 += kPartBatch * 64) {
        int col[kPartBatch];
        int2 r[kPartBatch];
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u) {
            const int i = min(s0 + u * 64 + lane, w.len - 1);
            col[u] = key[i] - first;
            r[u] = rec[i];
        }
#pragma unroll
        for (int u = 0; u < kPartBatch; ++u) {
            if (s0 + u * 64 >= w.len) break;
            const int c = col[u];
            const bool on = s0 + u * 64 + lane < w.len && c >= 0 && c < ncol;
            const uint32_t d = on ? (uint32_t)c : 0u;
            const unsigned long long m = same_digit(d, g.p.sub_shift, on);
            const uint32_t at = mine[d];
            const int before = bits_below(m);
            __builtin_amdgcn_wave_barrier();
            if (on && before == __popcll(m) - 1) mine[d] = at + (uint32_t)before + 1u;
            __builtin_amdgcn_wave_barrier();
            if (on) {
                if (sorted) {
                    s_out[at + before - origin] = r[u];
                } else {
                    g.t_colidx[at + before] = r[u].x;
                    if (g.t_vals) g.t_vals[at + before] = __int_as_float(r[u].y);
                }
            }
        }
    }
    if (!sorted) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < s_total; i += kPartThreads) {
        const int2 r = s_out[i];
        g.t_colidx[origin + i] = r.x;
        if (g.t_vals) g.t_vals[origin + i] = __int_as_float(r.y);
    }
}

static size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// An upper bound that grows with both arguments: a context whose buffers were sized for the largest graph it will see
// is bound to smaller ones as well, and the shape of a smaller relation may have more buckets than that of a larger one.
static size_t part_bytes(int64_t n_cols, int64_t nnz, bool records) {
    const size_t nb = (size_t)(n_cols < kMaxBuckets * 64 ? (n_cols + 63) / 64 : kMaxBuckets) + 64;
    const size_t tiles = (size_t)(nnz < (int64_t)kMinTile * kMaxTiles ? nnz / kMinTile + 1 : kMaxTiles);
    return align256(4 * tiles * nb) + align256(4 * nb) + align256(4 * (size_t)nnz) + (records ? align256(8 * (size_t)nnz) : 0) + 1024;
}

size_t csr_transpose_workspace(int64_t n_cols, int64_t nnz) { return part_bytes(n_cols, nnz, true); }

static void part_buffers(PartSeg& g, char* w) {
    g.hist = reinterpret_cast<uint32_t*>(w);
    w += align256(4 * (size_t)g.p.n_tiles * g.p.nb_pad);
    g.totals = reinterpret_cast<uint32_t*>(w);
    w += align256(4 * (size_t)g.p.nb_pad);
    g.key = reinterpret_cast<int32_t*>(w);
    w += align256(4 * (size_t)g.nnz);
    g.rec = reinterpret_cast<int2*>(w);
}

// Half the sets of counters where every relation of kMaxSub columns a workgroup has no more than two entries a column: clearing,
// adding up and rewriting the counters is most of the work there, and with 64 KB two workgroups fit a compute unit.  Transposes, all
// / half of the sets: 5 M columns, 1 M entries 143 / 91 us; 2 M columns with 1, 4, 6 and 8 M entries 68 / 52, 133 / 118, 186 / 180,
// 218 / 240; 1.2 M with 14 M 582 / 647.  A column that holds much of all entries makes its workgroup the last one, and half the
// wavefronts longer (4 M entries in 2 M columns, a third of them in one: 2.1 / 2.8 ms).
static bool few_per_column(const PartSeg& g) { return g.nnz <= 2 * (int64_t)g.n_cols; }

static int launch_partition(PartBatch& b, hipStream_t s) {
    int tiles = 0, scans = 0, cols = 0, nbp = 0, sub = 0;
    bool halve = true;
    for (int i = 0; i < b.n; ++i) {
        PartSeg& g = b.s[i];
        g.tile0 = tiles; g.scan0 = scans; g.col0 = cols;
        tiles += g.p.n_tiles;
        scans += g.p.nb_pad / 64;
        cols += (int)(((int64_t)g.n_cols + (int64_t(1) << g.p.sub_shift) - 1) >> g.p.sub_shift);
        if (g.p.nb_pad > nbp) nbp = g.p.nb_pad;
        if ((1 << g.p.sub_shift) > sub) sub = 1 << g.p.sub_shift;
        halve = halve && (1 << g.p.sub_shift < kMaxSub || few_per_column(g));
    }
    if (b.n == 0) return DR_OK;
    // Buckets hold 2048 to 4096 entries on average unless there are too many columns for that (kMaxBuckets); 5120 leave room
    // for their spread, and with the counters of 512 columns two workgroups fit a compute unit.
    const int sort_cap = sub <= kMaxSub / 2 ? 5120 : 0;
    const size_t lds3 = scatter_lds(nbp), lds4 = 4 * (size_t)kPartWaves * (halve && sub == kMaxSub ? sub / 2 : sub) + 8 * (size_t)sort_cap;
    static PerDevice raised;
    int dev = 0, lds_max = 0;
    DRC_HIP(hipGetDevice(&dev));
    DRC_TRY(raised.get(dev, &lds_max, [](int* n) -> int {    // all pass 64 KB, the last by its static words
        *n = 4 * kPartWaves * kMaxSub;
        DRC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&part_scatter_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)scatter_lds(kMaxBuckets)));
        DRC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&part_columns_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, *n));
        DRC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&part_columns_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, *n / 2));
        return DR_OK;
    }));
    hipLaunchKernelGGL(part_count_kernel, dim3((unsigned)tiles), dim3(kPartThreads), 0, s, b);
    hipLaunchKernelGGL(part_scan_kernel, dim3((unsigned)scans), dim3(1024), 0, s, b);
    if (b.s[0].count_only) hipLaunchKernelGGL((part_scatter_kernel<false>), dim3((unsigned)tiles), dim3(kPartThreads), lds3, s, b);
    else hipLaunchKernelGGL((part_scatter_kernel<true>), dim3((unsigned)tiles), dim3(kPartThreads), lds3, s, b);
    if (halve && sub == kMaxSub) hipLaunchKernelGGL((part_columns_kernel<true>), dim3((unsigned)cols), dim3(kPartThreads), lds4, s, b, sort_cap);
    else hipLaunchKernelGGL((part_columns_kernel<false>), dim3((unsigned)cols), dim3(kPartThreads), lds4, s, b, sort_cap);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_csr_transposes(const TransposeJob* jobs, int n, hipStream_t s) {
    PartBatch b{};
    for (int i = 0; i < n; ++i) {
        const TransposeJob& j = jobs[i];
        if (j.A->nnz == 0 || j.A->n_cols == 0) {
            DRC_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(j.t_rowptr), (size_t)j.A->n_cols + 1, 0u, s));
            continue;
        }
        PartSeg& g = b.s[b.n++];
        g.p = part_shape(j.A->n_cols, j.A->nnz);
        g.rowptr = j.A->rowptr; g.colidx = j.A->colidx; g.vals = j.A->vals;
        g.n_rows = (int)j.A->n_rows; g.n_cols = (int)j.A->n_cols; g.nnz = (int)j.A->nnz;
        g.t_rowptr = j.t_rowptr; g.t_colidx = j.t_colidx; g.t_vals = j.t_vals;
        part_buffers(g, static_cast<char*>(j.ws));
        if (b.n == kMaxPartSegs) {
            DRC_TRY(launch_partition(b, s));
            b = PartBatch{};
        }
    }
    return launch_partition(b, s);
}

// Up to so many entries the columns are counted with atomics: two launches before the one that writes the values, against the
// four of the partition.  Whole call, counted with atomics / by the partition: 20 000 entries 13 / 27 us, 200 000 16 / 31,
// 400 000 25 / 33, 800 000 45 / 34.
constexpr int64_t kCountByAtomics = 1 << 19;
// Symmetric normalisation: workspace = column counts | buffers of the partition.
size_t csr_normalize_workspace(int mode, int64_t n_cols, int64_t nnz) {
    if (mode != DR_NORM_SYM) return 0;
    return align256(4 * (size_t)(n_cols + 1)) + part_bytes(n_cols, nnz, false);
}

int launch_csr_normalize(int mode, int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t* rowptr,
                         const int32_t* colidx, float* vals_out, void* ws, hipStream_t s) {
    int32_t* deg_out = static_cast<int32_t*>(ws);
    if (mode == DR_NORM_SYM && nnz <= kCountByAtomics) {
        DRC_TRY(launch_count_columns(colidx, n_cols, nnz, deg_out, s));
    } else if (mode == DR_NORM_SYM) {
        PartBatch b{};
        PartSeg& g = b.s[b.n++];
        g.p = part_shape(n_cols, nnz);
        g.rowptr = rowptr; g.colidx = colidx;
        g.n_rows = (int)n_rows; g.n_cols = (int)n_cols; g.nnz = (int)nnz;
        g.t_rowptr = deg_out;
        g.count_only = 1;
        part_buffers(g, static_cast<char*>(ws) + align256(4 * (size_t)(n_cols + 1)));
        DRC_TRY(launch_partition(b, s));
    }
    return launch_normalize_kernel(mode, n_rows, nnz, rowptr, colidx, deg_out, vals_out, s);
}

}  // namespace drc
