// DR-SpMM forward (paper Section 3.2 / Alg. 1) and backward (Section 3.3 / Alg. 2).
//
// Work decomposition (both directions).  A wavefront owns RW consecutive CSR rows; the four wavefronts of a workgroup
// work independently except on very long rows, and the hardware dispatcher balances the (uneven) workgroups.
//   * The wavefront is split into 8 groups of 8 lanes; a group owns one row at a time and walks that
//     row's edges in storage order, so 8 rows are in flight per wavefront (the wave64 counterpart of the
//     paper's "partition the warp into parts, one neighbour each") and every row sum has one fixed
//     order: results are reproducible bit for bit.
//   * The wavefront's rows are ranked by degree, longest first, and a group that finishes a row takes the
//     next undealt one (a counter in LDS): the long rows start early, the short ones fill the gaps, and
//     the per-group totals come out balanced -- the paper's degree classes, resolved per block at run
//     time.  Which group sums a row does not change the order of that row's sum.
//   * Rows with more than kSolo edges are not given to one group: all 8 groups stride over their edges
//     into per-group partial sums that are then added in a fixed order (the tail of the power-law `near` degrees).
//   * Rows with more than kLong edges (high-fanout nets) are left to the end and then walked by all 32 groups of the
//     workgroup: one wavefront alone takes some 20 us per thousand edges, which on a 250 000-cell graph was as long as
//     all the rest of the launch (0.127 ms with 180 such nets against 0.064 ms for the relation's transpose, k = 8).
//   * Edge records (source column, edge value) are staged into LDS in sorted-row order with independent
//     coalesced loads.  A group then consumes its rows as ONE stream of records across row boundaries,
//     so the gather pipeline never drains between rows (rows have only a handful of edges).
//   * Gathers are issued in two ping-pong batches of a few edges per group: while one batch is being
//     accumulated the other is in flight, and no load in the loop is conditional (exhausted lanes gather
//     a valid dummy row), which lets the compiler wait on exactly the older batch.  The batch depth is
//     chosen per k so that a wavefront stays within 80 to 96 VGPRs and five wavefronts fit a SIMD: these
//     kernels wait on memory most of the time, and the number of wavefronts that can take turns matters
//     more than the depth of one wavefront's own pipeline (measured: 4 -> 6 wavefronts per SIMD, -3 %
//     of the whole layer step).
//   * Workgroup ids are remapped so each XCD walks a contiguous range of row blocks: neighbouring rows of
//     the spatially local `near` relation gather overlapping source rows, which then hit in that XCD's L2.
//   * One launch serves several relations (and several sub-graphs): the workgroups of an XCD take its share of the first
//     relation's blocks, then of the next one's.  Small relations fill the chip together instead of one after the other.
//
//   * Cache policy: what is read or written exactly once (the CSR records, the saved-index window, the
//     dense output rows) uses non-temporal loads and stores, so that the streams do not evict the gathered
//     rows from L2 and the memory-side cache (the forward output alone is 3-4x the gathered array); the
//     gathers themselves use the default policy.  Measured: -19 % on a random relation, -8 % on `near`.
//
// Forward.  Lane t of a group loads pairs [t*k/8, (t+1)*k/8) of the gathered source row with vector
// loads (one 128-byte line of values per source row at k = 32) and adds a*v into the group's private
// LDS row buffer with plain read-modify-write: the pairs of one source row have distinct columns and
// no other group touches the buffer, so no atomics are needed (ds_add_f32 runs at about 1/40 of the
// plain LDS rate on this chip).  A finished row goes to HBM in 128-byte segments.
//
// Backward.  Lane t of a group owns the compact outputs t, t+8, t+16, ... of its source row and keeps
// them in registers; per edge it reads dH[destination, idx[slot]] directly (the interleaved slot
// assignment keeps the 8 lanes of one load inside one 128-byte line of the dH row when 4k = D).
// In the layer the backward also finishes the input gradient (DENSE): a row's edges may come from two transposed
// relations behind one another (near and pins, both with cells as sources), the compact self-term gradient enters as one
// more record of the row, between the two lists, read like a gathered row, and the finished row is written once, dense, zero outside its
// selection.  Separate kernels wrote the compact sums, read them back (per relation) and wrote the dense rows.
#include "dr_internal.h"

namespace drc {

constexpr int kLPE = 8;          // lanes per row group
constexpr int kNG = kWave / kLPE;  // groups per wavefront
constexpr int kWPB = 4;          // wavefronts per workgroup
constexpr int kSolo = 32;        // rows with more edges are walked by all 8 groups of the wavefront together
constexpr int kLong = 256;       // rows with more edges are walked by all wavefronts of the workgroup together
constexpr int kCap = 256;        // edge records staged in LDS per pass (rows never straddle passes); 2 KB keeps
                                 // a forward workgroup below 27 KB of LDS, i.e. six of them per CU
constexpr int kStageIters = kCap / kWave;
constexpr int kBufPad = 4;       // row buffers are D + 4 words apart: group g starts 4 banks after group g-1
constexpr unsigned kValid = 0x80000000u, kLast = 0x40000000u, kRowMask = 0x0000ffffu;

template <int RW> struct WavePlan {
    int* sRp;      // [RW + 1] row pointers of the wavefront's rows
    int* sRp2;     // [RW + 1] the same in the second list (DENSE)
    int* sOrder;   // [RW]     slot -> local row; solo rows by degree, descending
    int* sStart;   // [RW + 1] slot -> offset of the row's records in sorted-row order
    int2* sRec;    // [kCap]   staged (column, value bits) records
    int* sNext;    // [1]      next undealt slot of the current pass
    int n_solo;
    unsigned long long coop_mask, zero_mask, long_mask;
};

template <int RW, bool DENSE = false> __host__ __device__ constexpr int plan_ints() {
    return 2 * kCap + (RW + 1) + RW + (RW + 1) + 2 + (DENSE ? RW + 2 : 0);      // even
}

// Orders the LDS accesses of one wavefront for the compiler (the hardware keeps them in program order).
__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// DENSE: rowptr may be null (no first list); rowptr2: second list of every row (may be null); extra: 1 if every row has one more record behind its lists
template <int RW, bool DENSE = false>
__device__ __forceinline__ WavePlan<RW> make_plan(int* base, const int32_t* __restrict__ rowptr, int r0, int nr,
                                                  const int32_t* __restrict__ rowptr2 = nullptr, int extra = 0) {
    WavePlan<RW> p;
    p.sRec = reinterpret_cast<int2*>(base);
    p.sRp = base + 2 * kCap;
    p.sOrder = p.sRp + (RW + 1);
    p.sStart = p.sOrder + RW;
    p.sNext = p.sStart + (RW + 1);

    const int lane = threadIdx.x & (kWave - 1);
    const bool have = !DENSE || rowptr != nullptr;
    const int rp_lo = have ? rowptr[r0 + min(lane, nr)] : 0;
    const int rp_hi = have ? rowptr[r0 + min(lane + 1, nr)] : 0;
    if (lane <= nr) p.sRp[lane] = rp_lo;
    int deg = (lane < nr) ? (rp_hi - rp_lo) : -1;
    bool solo = deg >= 1 && deg <= kSolo;
    if constexpr (DENSE) {
        p.sRp2 = p.sNext + 2;
        const int lo2 = rowptr2 ? rowptr2[r0 + min(lane, nr)] : 0, hi2 = rowptr2 ? rowptr2[r0 + min(lane + 1, nr)] : 0;
        if (lane <= nr) p.sRp2[lane] = lo2;
        const int tail = hi2 - lo2 + extra;       // either part of the row may be solo-sized: 2 * kSolo records fit a pass
        solo = lane < nr && deg <= kSolo && tail <= kSolo && deg + tail >= 1;
        deg += (lane < nr) ? tail : 0;
    }
    p.long_mask = __ballot(deg > kLong);
    p.coop_mask = __ballot(!solo && deg >= 1 && deg <= kLong);
    p.zero_mask = __ballot(deg == 0);
    p.n_solo = __popcll(__ballot(solo));
    // rank of every solo row among the solo rows: degree descending, row ascending
    const int key = solo ? deg : -1;
    int rank = 0;
#pragma unroll
    for (int j = 0; j < RW; ++j) {
        const int kj = __shfl(key, j, kWave);
        rank += (kj > key || (kj == key && j < lane)) ? 1 : 0;
    }
    if (solo) {
        p.sOrder[rank] = lane;
        p.sStart[rank] = deg;
    }
    lds_fence();
    const int x = (lane < p.n_solo) ? p.sStart[lane] : 0;
    int incl = x;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int y = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += y;
    }
    lds_fence();
    if (lane <= p.n_solo) p.sStart[lane] = incl - x;     // exclusive prefix; entry n_solo = total
    lds_fence();
    return p;
}

// End slot of the pass that starts at slot sa: as many whole solo rows as fit kCap records (at least one).
template <int RW> __device__ __forceinline__ int pass_end(const WavePlan<RW>& p, int sa) {
    const int lane = threadIdx.x & (kWave - 1);
    const int base = p.sStart[sa];
    const bool fits = lane > sa && lane <= p.n_solo && p.sStart[min(lane, p.n_solo)] - base <= kCap;
    return sa + __popcll(__ballot(fits));
}

// Stages the records of solo slots [sa, sb) into sRec, laid out in slot order.  Every lane issues its
// loads (at most kStageIters, all independent) before the first one is consumed.
// With `ecls` (adaptive-K backward) the degree class of the edge's other end point, one byte per stored entry,
// travels in the two top bits of the staged column (columns stay below 2^30 there).
constexpr unsigned kColMask = 0x3fffffffu;
__device__ __forceinline__ int tag_class(int col, const uint8_t* __restrict__ ecls, int e) {
    return ecls ? (col | ((int)__builtin_nontemporal_load(ecls + e) << 30)) : col;
}

// Where the records of a row come from.
struct RecSrc {
    const int32_t* colidx;
    const float* avals;
    const uint8_t* ecls;
    const int32_t* colidx2;       // second list (DENSE): its columns are shifted by col2_off
    const float* avals2;
    int col2_off, has_self;       // has_self: the row's own compact piece comes between the lists
};
struct RowSpan { int b1, d1, b2, d2; };      // first entry and number of entries in either list
constexpr uint32_t kSelfRec = 0xffffffffu;   // column of the record that stands for the row's own compact piece

template <int RW, bool DENSE> __device__ __forceinline__ RowSpan span_of(const WavePlan<RW>& p, int row) {
    RowSpan r{p.sRp[row], p.sRp[row + 1] - p.sRp[row], 0, 0};
    if constexpr (DENSE) { r.b2 = p.sRp2[row]; r.d2 = p.sRp2[row + 1] - p.sRp2[row]; }
    return r;
}

template <bool DENSE> __device__ __forceinline__ int2 fetch_rec(const RecSrc& s, const RowSpan& r, int off) {
    if constexpr (!DENSE) {
        const int e = r.b1 + off;
        return make_int2(tag_class(__builtin_nontemporal_load(s.colidx + e), s.ecls, e),
                         __float_as_int(__builtin_nontemporal_load(s.avals + e)));
    } else {
        // first list, own piece, second list: the order in which the same sums are formed when the first relation is
        // summed onto the own piece by the staged kernel, so that both ways give the same bits
        int2 rec = make_int2((int)kSelfRec, __float_as_int(1.0f));
        const bool second = off >= r.d1 + s.has_self;
        if (off < r.d1 || second) {
            const int e = second ? r.b2 + off - r.d1 - s.has_self : r.b1 + off;
            rec.x = __builtin_nontemporal_load((second ? s.colidx2 : s.colidx) + e) + (second ? s.col2_off : 0);
            rec.y = __float_as_int(__builtin_nontemporal_load((second ? s.avals2 : s.avals) + e));
        }
        return rec;
    }
}

template <bool DENSE, int RW>
__device__ __forceinline__ void stage_solo(const WavePlan<RW>& p, const RecSrc& src, int sa, int sb) {
    const int lane = threadIdx.x & (kWave - 1);
    const int base = p.sStart[sa];
    const int total = p.sStart[sb] - base;
    int2 r[kStageIters];
#pragma unroll
    for (int j = 0; j < kStageIters; ++j) {
        const int d = lane + kWave * j;
        const int dd = (d < total) ? d : 0;
        int lo = sa, hi = sb;                  // sStart[lo] - base <= dd < sStart[hi] - base
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (p.sStart[mid] - base <= dd) lo = mid; else hi = mid;
        }
        r[j] = fetch_rec<DENSE>(src, span_of<RW, DENSE>(p, p.sOrder[lo]), dd - (p.sStart[lo] - base));
    }
#pragma unroll
    for (int j = 0; j < kStageIters; ++j) {
        const int d = lane + kWave * j;
        if (d < total) p.sRec[d] = r[j];
    }
}

// Stages records [c0, c0 + n) of one long row (n <= kCap, n >= 1).
template <bool DENSE, int RW>
__device__ __forceinline__ void stage_chunk(const WavePlan<RW>& p, const RecSrc& src, const RowSpan& row, int c0, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    int2 r[kStageIters];
#pragma unroll
    for (int j = 0; j < kStageIters; ++j) {
        const int d = lane + kWave * j;
        r[j] = fetch_rec<DENSE>(src, row, c0 + ((d < n) ? d : 0));
    }
#pragma unroll
    for (int j = 0; j < kStageIters; ++j) {
        const int d = lane + kWave * j;
        if (d < n) p.sRec[d] = r[j];
    }
}

// Record stream of one group.  Solo mode: the group takes the next undealt row of the pass whenever it
// finishes one (rows are queued by degree, longest first, so the groups finish together), and consumes
// the records of its rows one after the other across row boundaries.
// Strided mode (long rows): records g, g + 8, ... of the staged chunk, no row boundaries.
struct Stream {
    int cur, row_end, row, done;
    // Every member is assigned on every path (selects, no branches): with a member written on one side of a branch
    // only, the compiler keeps the record in scratch memory and stores through a selected address, and a scratch
    // access is a vector-memory operation -- waiting for it drains the gathers in flight.
    template <int RW>
    __device__ __forceinline__ void take_slot(const WavePlan<RW>& p, int li, int sa, int npass, int base) {
        const bool ok = li < npass;
        const int s = sa + (ok ? li : 0);
        const int c = p.sStart[s] - base, e = p.sStart[s + 1] - base, r = p.sOrder[s];
        cur = ok ? c : cur;
        row_end = ok ? e : row_end;
        row = ok ? r : row;
        done = ok ? done : 1;
    }
    template <int RW>
    __device__ __forceinline__ void next_row(const WavePlan<RW>& p, int sa, int npass, int base) {
        const int lane = threadIdx.x & (kWave - 1);
        int li = 0;
        if ((lane & (kLPE - 1)) == 0) li = atomicAdd(p.sNext, 1);
        li = __shfl(li, lane & ~(kLPE - 1), kWave);
        take_slot(p, li, sa, npass, base);
    }
    // returns the meta word of the record just taken and advances
    template <bool STRIDED, int RW>
    __device__ __forceinline__ unsigned advance(const WavePlan<RW>& p, int sa, int npass, int base) {
        unsigned m = kValid | (unsigned)row;
        if constexpr (STRIDED) {
            cur += kNG;
            if (cur >= row_end) done = 1;
        } else {
            if (++cur == row_end) {
                m |= kLast;
                next_row(p, sa, npass, base);
            }
        }
        return m;
    }
};

// ---------------------------------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------------------------------

// The pairs of one gathered CBSR row that one lane of a group handles.
//   KPL > 0: KPL consecutive pairs [t*KPL, (t+1)*KPL), vector loads (k = 8*KPL).
//   KPL < 0: N = -KPL consecutive pairs as well, for every other k in (8*(N-1), 8*N]: lane t starts at pair N*t or, where
//            the row ends before N*t + N, at k - N.  Pairs a lower lane has got already are accumulated into the padding
//            words behind the row buffer, so no load or LDS access is conditional and none leaves the row.  Rows then
//            start at any multiple of 4 (values) or 2 (columns) bytes, which global loads of any width accept here.
//            Single pairs t, t+8, ... took 2 N loads an edge and lane in place of two to four: 45 677 x 100, k = 25, three
//            relations, D-ReLU and backward included 162 -> 155 us; a layer with one relation at k = 24, 223 -> 220 us.
template <int KPL> struct Pairs {
    static constexpr int N = KPL > 0 ? KPL : -KPL;
    float v[N];
    uint16_t c[N];
    // `k`: stored width of the row; `kk`: pairs of it that count (all, or a prefix of them in the adaptive-K kernels).
    // PREFIX: pairs at or past kk go to the padding words as well; where the lanes step back (KPL < 0) it is into the prefix, so
    // that what lies past it is not fetched (250 000 x 12 edges, D = 100, k = 25 with prefixes of 12 and 6: 184 -> 164 us; single pairs
    // took 166).
    template <bool PREFIX = false>
    __device__ __forceinline__ void load(const float* __restrict__ vals, const uint16_t* __restrict__ idx, uint32_t rowbase,
                                         int t, int k, int kk, int D) {
        const uint16_t padding = (uint16_t)(D + (t & (kBufPad - 1)));
        if constexpr (PREFIX && (KPL == -1 || KPL == -2)) {        // single pairs: as few loads, and the wide ones' masks spill
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int q = t + kLPE * u;
                const uint32_t off = rowbase + (uint32_t)min(q, kk - 1);
                v[u] = vals[off];
                const uint16_t col = idx[off];
                c[u] = q < kk ? col : padding;
            }
            return;
        }
        const int first = KPL > 0 ? KPL * t : min(N * t, PREFIX ? max(kk - N, 0) : k - N);
        load_raw(vals, idx, rowbase, t, first);
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (KPL < 0 ? first + u < N * t || (PREFIX && u > 0 && u >= kk)        // (the latter where the prefix is shorter than N)
                        : PREFIX && first + u >= kk) c[u] = padding;
    }
    __device__ __forceinline__ void load_raw(const float* __restrict__ vals, const uint16_t* __restrict__ idx, uint32_t rowbase,
                                             int t, int first) {
        if constexpr (KPL < 0) {
            const uint32_t off = rowbase + (uint32_t)first;
            __builtin_memcpy(v, vals + off, sizeof v);
            __builtin_memcpy(c, idx + off, sizeof c);
        } else if constexpr (KPL == 1) {
            v[0] = vals[rowbase + t];
            c[0] = idx[rowbase + t];
        } else if constexpr (KPL == 2) {
            const uint32_t off = rowbase + 2 * t;
            float2 a = *reinterpret_cast<const float2*>(vals + off);
            ushort2 b = *reinterpret_cast<const ushort2*>(idx + off);
            v[0] = a.x; v[1] = a.y; c[0] = b.x; c[1] = b.y;
        } else {
            const uint32_t off = rowbase + KPL * t;
#pragma unroll
            for (int q = 0; q < KPL / 4; ++q) {
                float4 a = *reinterpret_cast<const float4*>(vals + off + 4 * q);
                ushort4 b = *reinterpret_cast<const ushort4*>(idx + off + 4 * q);
                v[4 * q + 0] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
                c[4 * q + 0] = b.x; c[4 * q + 1] = b.y; c[4 * q + 2] = b.z; c[4 * q + 3] = b.w;
            }
        }
    }
    // buf[c] += a * v for all pairs; the columns of one CBSR row are distinct, so the reads can all be
    // issued before the writes (lanes past k share padding words: what lands there is never read)
    __device__ __forceinline__ void accumulate(float* buf, float a) const {
        float old[N];
#pragma unroll
        for (int u = 0; u < N; ++u) old[u] = buf[c[u]];
#pragma unroll
        for (int u = 0; u < N; ++u) buf[c[u]] = fmaf(a, v[u], old[u]);
    }
};

__device__ __forceinline__ void flush_row(float* __restrict__ out, float* buf, int D, int t, int vec_store) {
    if (vec_store) {
        for (int c = t * 4; c < D; c += kLPE * 4) {
            float4 v = *reinterpret_cast<const float4*>(buf + c);
            __builtin_nontemporal_store(v.x, out + c);          // merged into one 16-byte streaming store
            __builtin_nontemporal_store(v.y, out + c + 1);
            __builtin_nontemporal_store(v.z, out + c + 2);
            __builtin_nontemporal_store(v.w, out + c + 3);
            *reinterpret_cast<float4*>(buf + c) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else {
        for (int c = t; c < D; c += kLPE) {
            __builtin_nontemporal_store(buf[c], out + c);
            buf[c] = 0.0f;
        }
    }
}

template <int KPL, int EPI> struct FwdBatch {   // EPI consecutive stream records of one group, gathered
    Pairs<KPL> p[EPI];
    float a[EPI];
    unsigned meta[EPI];
};

// Degree classes of the adaptive-K variant (paper Section 3.2, Alg. 1 stage 2): a destination row with at most t1
// edges receives the k1 largest entries of each neighbour, one with at most t2 edges the k2 largest, the others k3.
struct DegreeK {
    int t1, t2, k2, k3;
    __device__ __forceinline__ int width(int deg, int k1) const { return deg <= t1 ? k1 : (deg <= t2 ? k2 : k3); }
    __device__ __forceinline__ int cls(int deg) const { return deg <= t1 ? 0 : (deg <= t2 ? 1 : 2); }
    __device__ __forceinline__ int width_of_class(int c, int k1) const { return c == 0 ? k1 : (c == 1 ? k2 : k3); }
};

template <int KPL, int EPI, bool STRIDED, bool ADAPT, int RW>
__device__ __forceinline__ void fwd_issue(FwdBatch<KPL, EPI>& b, Stream& st, const WavePlan<RW>& plan,
                                          const float* __restrict__ xs_vals, const uint16_t* __restrict__ xs_idx,
                                          int D, int k, int t, int g, int sa, int npass, int base, const DegreeK& dk) {
#pragma unroll
    for (int q = 0; q < EPI; ++q) {
        const bool valid = !st.done;
        const int2 rec = plan.sRec[valid ? st.cur : 0];
        const uint32_t col = valid ? (uint32_t)rec.x : 0u;   // exhausted lanes gather source row 0
        b.a[q] = __int_as_float(rec.y);
        int kk = k;                                          // pairs of the gathered row this destination takes
        // (strided: one row, whose width the caller has put into k1 and k2 = k3 = k1)
        if constexpr (ADAPT) kk = STRIDED ? dk.k3 : dk.width(plan.sRp[st.row + 1] - plan.sRp[st.row], k);   // a prefix of the rank order
        b.p[q].template load<ADAPT>(xs_vals, xs_idx, col * (uint32_t)k, t, k, kk, D);
        b.meta[q] = valid ? st.template advance<STRIDED, RW>(plan, sa, npass, base) : 0u;
    }
}

template <int KPL, int EPI>
__device__ __forceinline__ void fwd_consume(const FwdBatch<KPL, EPI>& b, float* buf, float* __restrict__ Hblk,
                                            int D, int t, int vec_store) {
#pragma unroll
    for (int q = 0; q < EPI; ++q) {
        if (b.meta[q] & kValid) {
            b.p[q].accumulate(buf, b.a[q]);
            if (b.meta[q] & kLast) flush_row(Hblk + (size_t)(b.meta[q] & kRowMask) * D, buf, D, t, vec_store);
        }
    }
}

template <int KPL, int EPI, bool STRIDED, bool ADAPT, int RW>
__device__ __forceinline__ void fwd_run(Stream& st, const WavePlan<RW>& plan, const float* __restrict__ xs_vals,
                                        const uint16_t* __restrict__ xs_idx, float* buf, float* __restrict__ Hblk,
                                        int D, int k, int t, int g, int sa, int npass, int base, int vec_store,
                                        const DegreeK& dk) {
    if constexpr (KPL != 0) {
        FwdBatch<KPL, EPI> A, B;
        fwd_issue<KPL, EPI, STRIDED, ADAPT, RW>(A, st, plan, xs_vals, xs_idx, D, k, t, g, sa, npass, base, dk);
        for (;;) {
            fwd_issue<KPL, EPI, STRIDED, ADAPT, RW>(B, st, plan, xs_vals, xs_idx, D, k, t, g, sa, npass, base, dk);
            fwd_consume(A, buf, Hblk, D, t, vec_store);
            if (!__any(B.meta[0] & kValid)) break;
            fwd_issue<KPL, EPI, STRIDED, ADAPT, RW>(A, st, plan, xs_vals, xs_idx, D, k, t, g, sa, npass, base, dk);
            fwd_consume(B, buf, Hblk, D, t, vec_store);
            if (!__any(A.meta[0] & kValid)) break;
        }
    } else {
        // k > 32 that is not 64 or 128: one record at a time, lane t takes pairs t, t+8, ... with scalar loads
        while (__any(!st.done)) {
            if (!st.done) {
                const int2 rec = plan.sRec[st.cur];
                const uint32_t rb = (uint32_t)rec.x * (uint32_t)k;
                const float a = __int_as_float(rec.y);
                for (int q = t; q < k; q += kLPE) {
                    const int c = xs_idx[rb + q];
                    buf[c] = fmaf(a, xs_vals[rb + q], buf[c]);
                }
                const unsigned m = st.template advance<STRIDED, RW>(plan, sa, npass, base);
                if (m & kLast) flush_row(Hblk + (size_t)(m & kRowMask) * D, buf, D, t, vec_store);
            }
        }
    }
}

struct SpmmFwdSeg {              // one relation of a launch
    const int32_t *rowptr, *colidx;
    const float *avals, *xs_vals;
    const uint16_t* xs_idx;
    float* H;
    int M, k, vec_store;
    int n_blocks, per_xcd, first;      // workgroups of this relation, per XCD, and where they start in an XCD's sequence
};
struct SpmmFwdArgs { SpmmFwdSeg s[kMaxSegs]; int n, D; };

// wavefronts per SIMD the registers are budgeted for (at D = 128 five of them fit the LDS as well)
constexpr int fwd_waves(int kpl, bool adapt) { return kpl == 16 || kpl == -8 ? 4 : (adapt || kpl < 0 || kpl > 1 ? 5 : 6); }

template <int KPL, int EPI, int RW, bool ADAPT>
__device__ __forceinline__ void spmm_fwd_rows(const SpmmFwdArgs& args, const DegreeK& dk) {
    static_assert(!ADAPT || KPL != 0, "the adaptive-K forward needs a path that can mask pairs");
    extern __shared__ float4 smem4[];
    __shared__ unsigned long long sLong[kWPB];
    const int local = blockIdx.x / kNumXcd, xcd = blockIdx.x % kNumXcd;
    int sg = 0;
    while (sg + 1 < args.n && local >= args.s[sg + 1].first) ++sg;
    const SpmmFwdSeg& s = args.s[sg];
    const int blk = xcd * s.per_xcd + local - s.first;
    if (blk >= s.n_blocks) return;
    const int32_t* __restrict__ rowptr = s.rowptr;
    const int32_t* __restrict__ colidx = s.colidx;
    const float* __restrict__ avals = s.avals;
    const float* __restrict__ xs_vals = s.xs_vals;
    const uint16_t* __restrict__ xs_idx = s.xs_idx;
    const int D = args.D, k = s.k, vec_store = s.vec_store;
    const RecSrc src{colidx, avals, nullptr, nullptr, nullptr, 0, 0};
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = min((blk * kWPB + wave) * RW, s.M);
    const int nr = min(RW, s.M - r0);
    const int g = lane / kLPE, t = lane % kLPE;
    const int ldb = D + kBufPad;
    const int wave_words = kNG * ldb + plan_ints<RW>();
    float* const base0 = reinterpret_cast<float*>(smem4);
    float* rowbuf = base0 + wave * wave_words;                       // [kNG][ldb], 16-byte aligned
    float* buf = rowbuf + g * ldb;
    float* Hblk = s.H + (size_t)r0 * D;

    for (int i = lane; i < kNG * ldb; i += kWave) rowbuf[i] = 0.0f;
    WavePlan<RW> plan = make_plan<RW>(reinterpret_cast<int*>(rowbuf + kNG * ldb), rowptr, r0, nr);
    if (lane == 0) sLong[wave] = plan.long_mask;
    __syncthreads();
    unsigned long long any_long = 0;
#pragma unroll
    for (int w = 0; w < kWPB; ++w) any_long |= sLong[w];

    // ---- rows without edges: zeros ----
    for (unsigned long long m = plan.zero_mask; m; m &= m - 1) {
        float* out = Hblk + (size_t)(__ffsll((long long)m) - 1) * D;
        for (int c = lane; c < D; c += kWave) __builtin_nontemporal_store(0.0f, out + c);
    }

    // ---- long rows: all groups stride over the row, partial sums added in a fixed order ----
    for (unsigned long long m = plan.coop_mask; m; m &= m - 1) {
        const int row = __ffsll((long long)m) - 1;
        const int e0 = plan.sRp[row], n = plan.sRp[row + 1] - e0;    // n <= kLong = kCap: one staged chunk
        DegreeK dkr = dk;
        if constexpr (ADAPT) dkr.k3 = dk.width(n, k);
        lds_fence();
        stage_chunk<false>(plan, src, RowSpan{e0, n, 0, 0}, 0, n);
        lds_fence();
        Stream st{g, n, row, g >= n ? 1 : 0};
        fwd_run<KPL, EPI, true, ADAPT, RW>(st, plan, xs_vals, xs_idx, buf, Hblk, D, k, t, g, 0, 0, 0, vec_store, dkr);
        lds_fence();
        float* out = Hblk + (size_t)row * D;
        for (int c = lane; c < D; c += kWave) {
            float sum = 0.0f;
#pragma unroll
            for (int q = 0; q < kNG; ++q) {
                sum += rowbuf[q * ldb + c];
                rowbuf[q * ldb + c] = 0.0f;
            }
            __builtin_nontemporal_store(sum, out + c);
        }
        lds_fence();
    }

    // ---- all other rows, in passes of at most kCap staged records ----
    for (int sa = 0; sa < plan.n_solo;) {
        const int sb = pass_end(plan, sa);
        lds_fence();
        if (lane == 0) *plan.sNext = kNG;
        stage_solo<false>(plan, src, sa, sb);
        lds_fence();
        Stream st{0, 0, 0, 0};
        st.take_slot(plan, g, sa, sb - sa, plan.sStart[sa]);     // first 8 rows of the pass: one per group
        fwd_run<KPL, EPI, false, ADAPT, RW>(st, plan, xs_vals, xs_idx, buf, Hblk, D, k, t, g, sa, sb - sa, plan.sStart[sa],
                                            vec_store, dk);
        sa = sb;
    }

    // ---- very long rows of the whole workgroup: each wavefront takes a quarter of the row ----
    if (!any_long) return;
    for (int w = 0; w < kWPB; ++w) {
        for (unsigned long long m = sLong[w]; m; m &= m - 1) {
            const int row = (blk * kWPB + w) * RW + __ffsll((long long)m) - 1;
            const int e0 = rowptr[row], e1 = rowptr[row + 1];
            DegreeK dkr = dk;
            if constexpr (ADAPT) dkr.k3 = dk.width(e1 - e0, k);
            const int per = (e1 - e0 + kWPB - 1) / kWPB;
            const int w0 = min(wave * per, e1 - e0), len = min(per, e1 - e0 - w0);      // lengths: sums may pass 2^31
            for (int c0 = 0; c0 < len; c0 += kCap) {
                const int n = min(kCap, len - c0);
                lds_fence();
                stage_chunk<false>(plan, src, RowSpan{e0 + w0 + c0, n, 0, 0}, 0, n);
                lds_fence();
                Stream st{g, n, 0, g >= n ? 1 : 0};
                fwd_run<KPL, EPI, true, ADAPT, RW>(st, plan, xs_vals, xs_idx, buf, Hblk, D, k, t, g, 0, 0, 0, vec_store, dkr);
            }
            __syncthreads();
            float* out = s.H + (size_t)row * D;
            for (int c = threadIdx.x; c < D; c += kWPB * kWave) {
                float sum = 0.0f;
                for (int q = 0; q < kWPB; ++q)
#pragma unroll
                    for (int p = 0; p < kNG; ++p) {
                        float* b = base0 + q * wave_words + p * ldb + c;
                        sum += *b;
                        *b = 0.0f;
                    }
                __builtin_nontemporal_store(sum, out + c);
            }
            __syncthreads();
        }
    }
}

template <int KPL, int EPI, int RW, bool ADAPT>
__global__ __launch_bounds__(kWPB * kWave, fwd_waves(KPL, ADAPT)) void spmm_fwd_kernel(SpmmFwdArgs args, DegreeK dk) {
    spmm_fwd_rows<KPL, EPI, RW, ADAPT>(args, dk);
}
template <int KPL, int EPI>
__global__ __launch_bounds__(kWPB * kWave, fwd_waves(KPL, false)) void spmm_fwd_mid_kernel(SpmmFwdArgs args, DegreeK dk) {
    spmm_fwd_rows<KPL, EPI, 16, false>(args, dk);
}

static int fwd_kind(const SpmmFwdJob& j) {
    const int k = j.k;
    int kpl = 0;
    if (k % kLPE == 0) {
        const int q = k / kLPE;
        if (q == 1) kpl = 1;
        else if (q == 2 && aligned(j.xs_vals, 8) && aligned(j.xs_idx, 4)) kpl = 2;
        else if ((q == 4 || q == 8 || q == 16) && aligned(j.xs_vals, 16) && aligned(j.xs_idx, 8)) kpl = q;
    }
    if (kpl == 0 && k <= 4 * kLPE) kpl = -((k + kLPE - 1) / kLPE);   // unaligned pairs
    return kpl;
}

template <int KPL, int EPI, bool ADAPT>
static void launch_fwd_kernel(SpmmFwdArgs& a, const LaunchShape& shape, DegreeK dk, hipStream_t s) {
    const int rw = ADAPT ? shape.forward_adaptive() : shape.forward(a.D);
    int first = 0;
    for (int i = 0; i < a.n; ++i) {
        SpmmFwdSeg& g = a.s[i];
        g.n_blocks = (g.M + kWPB * rw - 1) / (kWPB * rw);
        g.per_xcd = (g.n_blocks + kNumXcd - 1) / kNumXcd;
        g.first = first;
        first += g.per_xcd;
    }
    const dim3 grid((unsigned)(first * kNumXcd)), block(kWPB * kWave);
    const size_t buffers = sizeof(float) * kWPB * (size_t)kNG * (a.D + kBufPad), plan = sizeof(float) * kWPB;
    if (rw == 8) {
        hipLaunchKernelGGL((spmm_fwd_kernel<KPL, EPI, 8, ADAPT>), grid, block, buffers + plan * plan_ints<8>(), s, a, dk);
    } else if (rw == 32) {
        hipLaunchKernelGGL((spmm_fwd_kernel<KPL, EPI, 32, ADAPT>), grid, block, buffers + plan * plan_ints<32>(), s, a, dk);
    } else if constexpr (!ADAPT) {
        hipLaunchKernelGGL((spmm_fwd_mid_kernel<KPL, EPI>), grid, block, buffers + plan * plan_ints<16>(), s, a, dk);
    }
}

// Several relations at once: those whose width takes the same kernel share a launch.
int launch_spmm_fwds(const SpmmFwdJob* jobs, int n, int D, hipStream_t s) {
    unsigned long long done = 0;
    for (int i = 0; i < n; ++i) {
        if (done >> i & 1) continue;
        const SpmmFwdJob& j = jobs[i];
        if (j.A->n_rows == 0) continue;
        if (j.A->nnz == 0) {
            DRC_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(j.H), (size_t)j.A->n_rows * D, 0u, s));
            continue;
        }
        const int kind = fwd_kind(j);
        SpmmFwdArgs a{};
        a.D = D;
        LaunchShape shape;
        for (int r = i; r < n && a.n < kMaxSegs; ++r) {
            const SpmmFwdJob& q = jobs[r];
            if ((done >> r & 1) || q.A->nnz == 0 || fwd_kind(q) != kind) continue;
            done |= 1ull << r;
            shape.add(q.A->n_rows, q.A->n_cols, q.A->nnz);
            SpmmFwdSeg& g = a.s[a.n++];
            g = SpmmFwdSeg{q.A->rowptr, q.A->colidx, q.A->vals, q.xs_vals, q.xs_idx, q.H, (int)q.A->n_rows, q.k,
                           (D % 4 == 0 && aligned(q.H, 16)) ? 1 : 0, 0, 0, 0};
        }
        switch (kind) {
            case 1: launch_fwd_kernel<1, 4, false>(a, shape, DegreeK{}, s); break;
            case 2: launch_fwd_kernel<2, 3, false>(a, shape, DegreeK{}, s); break;
            case 4: launch_fwd_kernel<4, 2, false>(a, shape, DegreeK{}, s); break;
            case 8: launch_fwd_kernel<8, 1, false>(a, shape, DegreeK{}, s); break;
            case 16: launch_fwd_kernel<16, 1, false>(a, shape, DegreeK{}, s); break;
            case -1: launch_fwd_kernel<-1, 4, false>(a, shape, DegreeK{}, s); break;
            case -2: launch_fwd_kernel<-2, 3, false>(a, shape, DegreeK{}, s); break;
            case -3: launch_fwd_kernel<-3, 2, false>(a, shape, DegreeK{}, s); break;
            case -4: launch_fwd_kernel<-4, 2, false>(a, shape, DegreeK{}, s); break;
            default: launch_fwd_kernel<0, 1, false>(a, shape, DegreeK{}, s); break;
        }
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_spmm_fwd(const dr_csr* A, const float* xs_vals, const uint16_t* xs_idx, int D, int k, float* H, hipStream_t s) {
    const SpmmFwdJob j{A, xs_vals, xs_idx, k, H};
    return launch_spmm_fwds(&j, 1, D, s);
}

int launch_spmm_fwd_adaptive(const dr_csr* A, const float* xr_vals, const uint16_t* xr_idx, int D, const dr_degree_classes* c,
                             float* H, hipStream_t s) {
    const int k = c->k1;
    if (A->nnz == 0) return launch_fill_u32(reinterpret_cast<uint32_t*>(H), (size_t)A->n_rows * D, 0u, s);
    const DegreeK dk{c->t1, c->t2, c->k2, c->k3};
    SpmmFwdArgs a{};
    a.D = D;
    a.n = 1;
    LaunchShape shape;
    shape.add(A->n_rows, A->n_cols, A->nnz);
    a.s[0] = SpmmFwdSeg{A->rowptr, A->colidx, A->vals, xr_vals, xr_idx, H, (int)A->n_rows, k, (D % 4 == 0 && aligned(H, 16)) ? 1 : 0, 0, 0, 0};
    // widths that fill the lanes evenly keep the vector loads of the uniform kernel (pairs past the destination's
    // width are redirected after the load); the others take unaligned pairs
    const bool vec = (k == 8) || (k == 16 && aligned(xr_vals, 8) && aligned(xr_idx, 4)) ||
                     ((k == 32 || k == 64) && aligned(xr_vals, 16) && aligned(xr_idx, 8));
    switch (vec ? k / kLPE + 100 : (k + kLPE - 1) / kLPE) {
        case 101: launch_fwd_kernel<1, 4, true>(a, shape, dk, s); break;
        case 102: launch_fwd_kernel<2, 3, true>(a, shape, dk, s); break;
        case 104: launch_fwd_kernel<4, 2, true>(a, shape, dk, s); break;
        case 108: launch_fwd_kernel<8, 1, true>(a, shape, dk, s); break;
        case 1: launch_fwd_kernel<-1, 4, true>(a, shape, dk, s); break;
        case 2: launch_fwd_kernel<-2, 3, true>(a, shape, dk, s); break;
        case 3: launch_fwd_kernel<-3, 2, true>(a, shape, dk, s); break;
        case 4: launch_fwd_kernel<-4, 2, true>(a, shape, dk, s); break;
        default: launch_fwd_kernel<-8, 1, true>(a, shape, dk, s); break;   // k1 <= 64 (checked by the caller)
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

// ---------------------------------------------------------------------------------------------------
// backward: rows are sources j (rows of A^T); lane t of the row's group owns compact slots
// s0 + t, s0 + t + 8, ... (KPL of them) in registers.  k larger than 8*KPL is covered by re-walking the
// block for the next window of slots.
// ---------------------------------------------------------------------------------------------------

template <int KPL, int EPI> struct BwdBatch {
    float v[EPI][KPL];
    float a[EPI];
    unsigned meta[EPI];
};

// A staged saved column carries a flag in its top bit (columns are below 2^15): the slot's gradient is gated off.
constexpr unsigned kIdxMask = 0x7fffu, kGateOff = 0x8000u;

// saved columns of the slots lane t owns; ci[KPL] (one extra word) = column of the row's slot 0, which the
// adaptive-K kernel reads in place of the slots a destination does not take
template <int KPL, bool DENSE>
__device__ __forceinline__ void load_ci(int (&ci)[KPL + 1], const uint16_t* sIdx, int row, int t) {
#pragma unroll
    for (int u = 0; u < KPL; ++u) ci[u] = sIdx[row * (kLPE * KPL) + t + kLPE * u] & (DENSE ? kIdxMask : 0xffffu);
    ci[KPL] = sIdx[row * (kLPE * KPL)] & (DENSE ? kIdxMask : 0xffffu);
}

constexpr unsigned kClassShift = 16;   // adaptive-K backward: degree class of the record's destination in meta bits 16-17

// What DENSE adds: the rows' own compact pieces (rowbase: row number of local row 0).
struct SelfPiece { const float* init; int rowbase; };

template <int KPL, int EPI, bool STRIDED, bool ADAPT, bool DENSE, int RW>
__device__ __forceinline__ void bwd_issue(BwdBatch<KPL, EPI>& b, Stream& st, int (&ci)[KPL + 1], const WavePlan<RW>& plan,
                                          const uint16_t* sIdx, const float* __restrict__ dH, int D, int k, int t, int g,
                                          int sa, int npass, int base, const DegreeK& dk, const SelfPiece& self) {
#pragma unroll
    for (int q = 0; q < EPI; ++q) {
        const bool valid = !st.done;
        const int2 rec = plan.sRec[valid ? st.cur : 0];
        uint32_t col = valid ? (uint32_t)rec.x : 0u;
        const bool own = DENSE && col == kSelfRec;
        unsigned cls = 0;
        if constexpr (ADAPT) { cls = col >> 30; col &= kColMask; }
        b.a[q] = __int_as_float(rec.y);
        const float* rowp = dH + (size_t)col * (uint32_t)D;
        if constexpr (ADAPT) {
            // slots at or past the destination's width read the column of slot 0 instead (a word the group's first
            // lane reads anyway): no load is conditional, and no further sector of the dH row is touched
            const int kq = dk.width_of_class((int)cls, k);
#pragma unroll
            for (int u = 0; u < KPL; ++u) b.v[q][u] = rowp[(t + kLPE * u < kq) ? ci[u] : ci[KPL]];
        } else if constexpr (DENSE) {
            const float* p = own ? self.init + (size_t)(self.rowbase + st.row) * (uint32_t)k : rowp;
#pragma unroll
            for (int u = 0; u < KPL; ++u) b.v[q][u] = p[own ? min(t + kLPE * u, k - 1) : ci[u]];
        } else {
#pragma unroll
            for (int u = 0; u < KPL; ++u) b.v[q][u] = rowp[ci[u]];
        }
        unsigned m = 0;
        if (valid) {
            m = st.template advance<STRIDED, RW>(plan, sa, npass, base) | (cls << kClassShift);
            if (!STRIDED && (m & kLast) && !st.done) load_ci<KPL, DENSE>(ci, sIdx, st.row, t);
        }
        b.meta[q] = m;
    }
}

// Further pieces and output of a dense row: out[row, :] = rowbuf, plus a second compact piece at its own columns.
struct DenseOut {
    float* out;              // [N, D]
    const CompactPiece* more;    // [2] further pieces at selections of their own (idx null: none)
    int D;
    float* rowbuf;           // [D] LDS, zero between rows
    const uint16_t* sIdx;
};

// rowbuf holds the row's own values; called by a whole wavefront
__device__ __forceinline__ void emit_row(const DenseOut& o, size_t row, int lane) {
    lds_fence();
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const CompactPiece& c = o.more[m];
        if (!c.idx) continue;
        for (int q = lane; q < c.k; q += kWave) {           // the columns of one selection are distinct
            const size_t at = row * c.k + q;
            o.rowbuf[c.idx[at]] += (c.gate && !(c.gate[at] > 0.0f)) ? 0.0f : c.vals[at];
        }
        lds_fence();
    }
    float* p = o.out + row * o.D;
    for (int c = 2 * lane; c < o.D; c += 2 * kWave) {       // D is a multiple of 32
        const float2 v = *reinterpret_cast<const float2*>(o.rowbuf + c);
        __builtin_nontemporal_store(v.x, p + c);
        __builtin_nontemporal_store(v.y, p + c + 1);
        *reinterpret_cast<float2*>(o.rowbuf + c) = make_float2(0.f, 0.f);
    }
    lds_fence();
}

template <int KPL, int EPI, bool ADAPT, bool DENSE>
__device__ __forceinline__ void bwd_consume(const BwdBatch<KPL, EPI>& b, float (&acc)[KPL], float* __restrict__ Gblk,
                                            int k, int s0, int t, int accumulate, const DegreeK& dk, const DenseOut& dense, int r0) {
#pragma unroll
    for (int q = 0; q < EPI; ++q) {
        if (b.meta[q] & kValid) {
            if constexpr (ADAPT) {
                const int kq = dk.width_of_class((int)((b.meta[q] >> kClassShift) & 3u), k);
#pragma unroll
                for (int u = 0; u < KPL; ++u) acc[u] = fmaf(b.a[q], (t + kLPE * u < kq) ? b.v[q][u] : 0.f, acc[u]);
            } else {
#pragma unroll
                for (int u = 0; u < KPL; ++u) acc[u] = fmaf(b.a[q], b.v[q][u], acc[u]);
            }
            if (!DENSE && (b.meta[q] & kLast)) {
                float* o = Gblk + (size_t)(b.meta[q] & kRowMask) * k;
#pragma unroll
                for (int u = 0; u < KPL; ++u) {
                    const int slot = s0 + t + kLPE * u;
                    if (slot < k) o[slot] = accumulate ? (o[slot] + acc[u]) : acc[u];
                    acc[u] = 0.f;
                }
            }
        }
        if constexpr (DENSE) {
            // finished rows of this record, one after the other: the group scatters its slots, the wavefront writes the row
            const int lane = threadIdx.x & (kWave - 1);
            unsigned long long last = __ballot((b.meta[q] & (kValid | kLast)) == (kValid | kLast));
            while (last) {
                const int src = __ffsll((long long)last) - 1;
                const int row = (int)((unsigned)__builtin_amdgcn_readlane((int)b.meta[q], src) & kRowMask);
                if ((lane / kLPE) == (src / kLPE)) {
#pragma unroll
                    for (int u = 0; u < KPL; ++u) {
                        const unsigned c = dense.sIdx[row * (kLPE * KPL) + t + kLPE * u];
                        if (t + kLPE * u < k) dense.rowbuf[c & kIdxMask] = (c & kGateOff) ? 0.0f : acc[u];
                        acc[u] = 0.f;
                    }
                }
                emit_row(dense, (size_t)(r0 + row), lane);
                last &= ~(0xffull << (src & ~(kLPE - 1)));
            }
        }
    }
}

template <int KPL, int EPI, bool STRIDED, bool ADAPT, bool DENSE, int RW>
__device__ __forceinline__ void bwd_run(Stream& st, int (&ci)[KPL + 1], float (&acc)[KPL], const WavePlan<RW>& plan,
                                        const uint16_t* sIdx, const float* __restrict__ dH, float* __restrict__ Gblk,
                                        int D, int k, int s0, int t, int g, int sa, int npass, int base,
                                        int accumulate, const DegreeK& dk, const SelfPiece& self, const DenseOut& dense) {
    constexpr bool kFlush = DENSE && !STRIDED;       // a strided row is put together from the groups' parts afterwards
    BwdBatch<KPL, EPI> A, B;
    bwd_issue<KPL, EPI, STRIDED, ADAPT, DENSE, RW>(A, st, ci, plan, sIdx, dH, D, k, t, g, sa, npass, base, dk, self);
    for (;;) {
        bwd_issue<KPL, EPI, STRIDED, ADAPT, DENSE, RW>(B, st, ci, plan, sIdx, dH, D, k, t, g, sa, npass, base, dk, self);
        bwd_consume<KPL, EPI, ADAPT, kFlush>(A, acc, Gblk, k, s0, t, accumulate, dk, dense, self.rowbase);
        if (!__any(B.meta[0] & kValid)) break;
        bwd_issue<KPL, EPI, STRIDED, ADAPT, DENSE, RW>(A, st, ci, plan, sIdx, dH, D, k, t, g, sa, npass, base, dk, self);
        bwd_consume<KPL, EPI, ADAPT, kFlush>(B, acc, Gblk, k, s0, t, accumulate, dk, dense, self.rowbase);
        if (!__any(A.meta[0] & kValid)) break;
    }
}

struct SpmmBwdSeg {              // the transposed relation (or pair of relations) of one kind of source rows
    const int32_t *rowptr, *colidx;
    const float *avals, *dH;
    const uint16_t* xs_idx;
    float* dXs;                  // compact [N, k], or (DENSE) dense [N, D]
    const uint8_t* ecls;
    int N, k, accumulate;
    int n_blocks, per_xcd, first;
    // DENSE
    const int32_t *rowptr2, *colidx2;
    const float *avals2, *init, *gate;
    CompactPiece more[2];
    int col2_off;
};
struct SpmmBwdArgs { SpmmBwdSeg s[kMaxSegs]; int n, D; };
static_assert(sizeof(SpmmBwdArgs) < 4096, "kernel arguments");

template <int KPL, int RW, bool DENSE> constexpr int bwd_wave_words(int D) {     // LDS words of one wavefront
    return kNG * kLPE * KPL + RW * kLPE * KPL / 2 + plan_ints<RW, DENSE>() + (DENSE ? D : 0);
}

// Partial sums of weight gradients, in workgroups behind those of the rows: 64 entries of one gradient each.  They need a few
// microseconds of loads one behind the other, which pass under the last rows; as a launch of their own they took 5 to 7
// (layers of 2 048 to 60 000 cells).  64 bits: up to 1024 partials (256 workgroups of 4 at D = 32) of nearly equal size lose as much in
// 32-bit sums as everything before.
constexpr int kSumEntries = kWave;
__device__ __forceinline__ void sum_partials(const PartialSum* __restrict__ table, int per, int block, double* sums) {
    const PartialSum p = table[block / per];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int at = (block % per) * kSumEntries + lane;
    const float* src = p.src + at;
    double s = 0.0;
    constexpr int U = 16;
    int b = wave;
    for (; b + (U - 1) * kWPB < p.n; b += U * kWPB) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = src[(size_t)(b + u * kWPB) * p.count];
#pragma unroll
        for (int u = 0; u < U; ++u) s += (double)v[u];
    }
    for (; b < p.n; b += 4 * kWPB) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = b + u * kWPB < p.n ? src[(size_t)(b + u * kWPB) * p.count] : 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) s += (double)v[u];
    }
    sums[wave * kWave + lane] = s;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 1; w < kWPB; ++w) s += sums[w * kWave + lane];
        p.dst[at] = (float)((double)kUnscale * s);
    }
}
constexpr size_t kSumLds = sizeof(double) * kWPB * kWave;
__global__ __launch_bounds__(kWPB * kWave) void pending_sums_kernel(const PartialSum* __restrict__ table, int per) {
    __shared__ double sums[kWPB * kWave];
    sum_partials(table, per, blockIdx.x, sums);
}
int launch_pending_sums(const PendingSums& pending, hipStream_t s) {
    if (pending.n == 0) return DR_OK;
    const int per = pending.count / kSumEntries;
    hipLaunchKernelGGL(pending_sums_kernel, dim3((unsigned)(pending.n * per)), dim3(kWPB * kWave), 0, s, pending.table, per);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

struct SumTail { const PartialSum* table; int first, per; };      // workgroups from `first` on; table null: none

template <int KPL, int EPI, int RW, bool ADAPT, bool DENSE>
__device__ __forceinline__ void spmm_bwd_rows(const SpmmBwdArgs& args, const DegreeK& dk, const SumTail& tail) {
    extern __shared__ float4 smem4[];
    __shared__ unsigned long long sLong[kWPB];
    constexpr int kWin = kLPE * KPL;                                       // compact slots per pass over the block
    if constexpr (DENSE) {
        if (tail.table && (int)blockIdx.x >= tail.first) {
            sum_partials(tail.table, tail.per, (int)blockIdx.x - tail.first, reinterpret_cast<double*>(smem4));
            return;
        }
    }
    const int local = blockIdx.x / kNumXcd, xcd = blockIdx.x % kNumXcd;
    int sg = 0;
    while (sg + 1 < args.n && local >= args.s[sg + 1].first) ++sg;
    const SpmmBwdSeg& s = args.s[sg];
    const int blk = xcd * s.per_xcd + local - s.first;
    if (blk >= s.n_blocks) return;
    const int32_t* __restrict__ t_rowptr = s.rowptr;
    const float* __restrict__ dH = s.dH;
    const uint16_t* __restrict__ xs_idx = s.xs_idx;
    const int D = args.D, k = s.k, accumulate = s.accumulate;
    const RecSrc src{s.colidx, s.avals, ADAPT ? s.ecls : nullptr, s.colidx2, s.avals2, s.col2_off, DENSE && s.init ? 1 : 0};
    const int kWords = bwd_wave_words<KPL, RW, DENSE>(D);
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* const base0 = reinterpret_cast<float*>(smem4);
    float* part = base0 + wave * kWords;                                   // [kNG][kWin] long-row partials
    uint16_t* sIdx = reinterpret_cast<uint16_t*>(part + kNG * kWin);       // [RW][kWin] saved columns of the window
    float* rowbuf = part + kNG * kWin + RW * kWin / 2 + plan_ints<RW, DENSE>();    // DENSE: [D]
    const int r0 = min((blk * kWPB + wave) * RW, s.N);
    const int nr = min(RW, s.N - r0);
    const int g = lane / kLPE, t = lane % kLPE;
    float* Gblk = s.dXs + (size_t)r0 * k;
    const SelfPiece self{s.init, r0};
    const DenseOut dense{s.dXs, s.more, D, rowbuf, sIdx};

    WavePlan<RW> plan = make_plan<RW, DENSE>(reinterpret_cast<int*>(part + kNG * kWin + RW * kWin / 2), t_rowptr, r0, nr,
                                             DENSE ? s.rowptr2 : nullptr, DENSE && s.init ? 1 : 0);
    if constexpr (DENSE)
        for (int c = lane; c < D; c += kWave) rowbuf[c] = 0.0f;
    if (lane == 0) sLong[wave] = plan.long_mask;
    __syncthreads();
    unsigned long long any_long = 0;
#pragma unroll
    for (int w = 0; w < kWPB; ++w) any_long |= sLong[w];

    for (int s0 = 0; s0 < (DENSE ? 1 : k); s0 += kWin) {         // DENSE: k <= kWin, one window
        // saved columns of this window for every row of the block (0 beyond k)
        lds_fence();
        for (int i = lane; i < nr * kWin; i += kWave) {
            const int row = i / kWin, w = i % kWin;
            const size_t at = (size_t)(r0 + row) * k + s0 + w;
            uint16_t c = (s0 + w < k) ? __builtin_nontemporal_load(xs_idx + at) : (uint16_t)0;
            if constexpr (DENSE)
                if (s.gate && w < k && !(__builtin_nontemporal_load(s.gate + at) > 0.0f)) c |= kGateOff;
            sIdx[i] = c;
        }
        lds_fence();

        // ---- rows without records ----
        if (DENSE || !accumulate) {
            for (unsigned long long m = plan.zero_mask; m; m &= m - 1) {
                const int row = __ffsll((long long)m) - 1;
                if constexpr (DENSE) {
                    emit_row(dense, (size_t)(r0 + row), lane);
                } else {
                    float* o = Gblk + (size_t)row * k;
                    for (int w = lane; w < kWin; w += kWave)
                        if (s0 + w < k) o[s0 + w] = 0.0f;
                }
            }
        }

        // ---- long rows ----
        for (unsigned long long m = plan.coop_mask; m; m &= m - 1) {
            const int row = __ffsll((long long)m) - 1;
            const RowSpan span = span_of<RW, DENSE>(plan, row);
            const int n = span.d1 + span.d2 + (DENSE && s.init ? 1 : 0);   // n <= kLong = kCap: one staged chunk
            int ci[KPL + 1];
            float acc[KPL];
            load_ci<KPL, DENSE>(ci, sIdx, row, t);
#pragma unroll
            for (int u = 0; u < KPL; ++u) acc[u] = 0.f;
            lds_fence();
            stage_chunk<DENSE>(plan, src, span, 0, n);
            lds_fence();
            Stream st{g, n, row, g >= n ? 1 : 0};
            bwd_run<KPL, EPI, true, ADAPT, DENSE, RW>(st, ci, acc, plan, sIdx, dH, Gblk, D, k, s0, t, g, 0, 0, 0, accumulate, dk, self, dense);
#pragma unroll
            for (int u = 0; u < KPL; ++u) part[g * kWin + t + kLPE * u] = acc[u];
            lds_fence();
            for (int w = lane; w < kWin; w += kWave) {
                if (s0 + w < k) {
                    float sum = 0.f;
#pragma unroll
                    for (int q = 0; q < kNG; ++q) sum += part[q * kWin + w];
                    if constexpr (DENSE) {
                        const unsigned c = sIdx[row * kWin + w];
                        rowbuf[c & kIdxMask] = (c & kGateOff) ? 0.0f : sum;
                    } else {
                        float* o = Gblk + (size_t)row * k + s0 + w;
                        *o = accumulate ? (*o + sum) : sum;
                    }
                }
            }
            if constexpr (DENSE) emit_row(dense, (size_t)(r0 + row), lane);
            lds_fence();
        }

        // ---- all other rows ----
        for (int sa = 0; sa < plan.n_solo;) {
            const int sb = pass_end(plan, sa);
            lds_fence();
            if (lane == 0) *plan.sNext = kNG;
            stage_solo<DENSE>(plan, src, sa, sb);
            lds_fence();
            Stream st{0, 0, 0, 0};
            st.take_slot(plan, g, sa, sb - sa, plan.sStart[sa]);
            int ci[KPL + 1];
            float acc[KPL];
            ci[KPL] = 0;
#pragma unroll
            for (int u = 0; u < KPL; ++u) { ci[u] = 0; acc[u] = 0.f; }
            if (!st.done) load_ci<KPL, DENSE>(ci, sIdx, st.row, t);
            bwd_run<KPL, EPI, false, ADAPT, DENSE, RW>(st, ci, acc, plan, sIdx, dH, Gblk, D, k, s0, t, g, sa, sb - sa, plan.sStart[sa],
                                                       accumulate, dk, self, dense);
            sa = sb;
        }

        // ---- very long rows of the whole workgroup: each wavefront takes a quarter of the row ----
        if (!any_long) continue;
        for (int w = 0; w < kWPB; ++w) {
            for (unsigned long long m = sLong[w]; m; m &= m - 1) {
                const int row = (blk * kWPB + w) * RW + __ffsll((long long)m) - 1;
                RowSpan span{0, 0, 0, 0};
                if (!DENSE || t_rowptr) { span.b1 = t_rowptr[row]; span.d1 = t_rowptr[row + 1] - span.b1; }
                if (DENSE && s.rowptr2) { span.b2 = s.rowptr2[row]; span.d2 = s.rowptr2[row + 1] - span.b2; }
                const int n_all = span.d1 + span.d2 + (DENSE && s.init ? 1 : 0);
                const int per = (n_all + kWPB - 1) / kWPB;
                const int w0 = min(wave * per, n_all), w1 = min(w0 + per, n_all);
                int ci[KPL + 1];
                float acc[KPL];
#pragma unroll
                for (int u = 0; u < KPL; ++u) {
                    const int slot = s0 + t + kLPE * u;
                    ci[u] = slot < k ? xs_idx[(size_t)row * k + slot] : 0;
                    acc[u] = 0.f;
                }
                ci[KPL] = xs_idx[(size_t)row * k];                          // (adaptive K: one window, s0 = 0)
                for (int c0 = w0; c0 < w1; c0 += kCap) {
                    const int n = min(kCap, w1 - c0);
                    lds_fence();
                    stage_chunk<DENSE>(plan, src, span, c0, n);
                    lds_fence();
                    Stream st{g, n, 0, g >= n ? 1 : 0};
                    bwd_run<KPL, EPI, true, ADAPT, DENSE, RW>(st, ci, acc, plan, sIdx, dH, Gblk, D, k, s0, t, g, 0, 0, 0, accumulate, dk,
                                                              SelfPiece{s.init, row}, dense);
                }
#pragma unroll
                for (int u = 0; u < KPL; ++u) part[g * kWin + t + kLPE * u] = acc[u];
                __syncthreads();
                if (wave == 0) {
                    for (int i = lane; i < kWin; i += kWave) {
                        if (s0 + i < k) {
                            float sum = 0.f;
                            for (int q = 0; q < kWPB; ++q)
#pragma unroll
                                for (int p = 0; p < kNG; ++p) sum += base0[q * kWords + p * kWin + i];
                            const size_t at = (size_t)row * k + s0 + i;
                            if constexpr (DENSE) {
                                rowbuf[xs_idx[at]] = (s.gate && !(s.gate[at] > 0.0f)) ? 0.0f : sum;
                            } else {
                                s.dXs[at] = accumulate ? (s.dXs[at] + sum) : sum;
                            }
                        }
                    }
                    if constexpr (DENSE) emit_row(dense, (size_t)row, lane);
                }
                __syncthreads();
            }
        }
    }
}

constexpr int bwd_waves(int kpl, bool adapt, bool dense) { return kpl == 8 ? 4 : (adapt || dense || kpl == 4 ? 5 : 6); }
template <int KPL, int EPI, int RW, bool ADAPT, bool DENSE>
__global__ __launch_bounds__(kWPB * kWave, bwd_waves(KPL, ADAPT, DENSE)) void spmm_bwd_kernel(SpmmBwdArgs args, DegreeK dk, SumTail tail) {
    spmm_bwd_rows<KPL, EPI, RW, ADAPT, DENSE>(args, dk, tail);
}
template <int KPL, int EPI, bool ADAPT, bool DENSE>
__global__ __launch_bounds__(kWPB * kWave, bwd_waves(KPL, ADAPT, DENSE)) void spmm_bwd_mid_kernel(SpmmBwdArgs args, DegreeK dk, SumTail tail) {
    spmm_bwd_rows<KPL, EPI, 16, ADAPT, DENSE>(args, dk, tail);
}

template <int KPL, int EPI, bool ADAPT, bool DENSE>
static void launch_bwd_kernel(SpmmBwdArgs& a, const LaunchShape& shape, DegreeK dk, hipStream_t s, const PendingSums& sums = PendingSums{}) {
    const int rw = DENSE ? shape.dense(a.D) : shape.compact(a.D);
    int first = 0;
    for (int i = 0; i < a.n; ++i) {
        SpmmBwdSeg& g = a.s[i];
        g.n_blocks = (g.N + kWPB * rw - 1) / (kWPB * rw);
        g.per_xcd = (g.n_blocks + kNumXcd - 1) / kNumXcd;
        g.first = first;
        first += g.per_xcd;
    }
    SumTail tail{nullptr, first * kNumXcd, 0};
    int extra = 0;
    if (DENSE && sums.n) {
        tail.table = sums.table;
        tail.per = sums.count / kSumEntries;
        extra = sums.n * tail.per;
    }
    const dim3 grid((unsigned)(first * kNumXcd + extra)), block(kWPB * kWave);
    const auto lds = [&](int words) {
        const size_t bytes = sizeof(float) * kWPB * (size_t)words;
        return extra && bytes < kSumLds ? kSumLds : bytes;
    };
    if (rw == 8) {
        hipLaunchKernelGGL((spmm_bwd_kernel<KPL, EPI, 8, ADAPT, DENSE>), grid, block, lds(bwd_wave_words<KPL, 8, DENSE>(a.D)), s, a, dk, tail);
    } else if (rw == 16) {
        hipLaunchKernelGGL((spmm_bwd_mid_kernel<KPL, EPI, ADAPT, DENSE>), grid, block, lds(bwd_wave_words<KPL, 16, DENSE>(a.D)), s, a, dk, tail);
    } else if constexpr (DENSE || KPL < 8) {      // (compact: rows of D <= 32 only, k <= 32 then)
        hipLaunchKernelGGL((spmm_bwd_kernel<KPL, EPI, 32, ADAPT, DENSE>), grid, block, lds(bwd_wave_words<KPL, 32, DENSE>(a.D)), s, a, dk, tail);
    }
}

static int bwd_kind(int k) { return k <= 8 ? 1 : (k <= 16 ? 2 : (k <= 32 ? 4 : 8)); }

// Several transposed relations at once (no job reads what another writes); equal kernels share a launch.
int launch_spmm_bwds(const SpmmBwdJob* jobs, int n, int D, hipStream_t s) {
    unsigned long long done = 0;
    for (int i = 0; i < n; ++i) {
        if (done >> i & 1) continue;
        const SpmmBwdJob& j = jobs[i];
        if (j.At->n_rows == 0) continue;
        if (j.At->nnz == 0) {
            if (!j.accumulate) DRC_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(j.dXs), (size_t)j.At->n_rows * j.k, 0u, s));
            continue;
        }
        const int kind = bwd_kind(j.k);
        SpmmBwdArgs a{};
        a.D = D;
        LaunchShape shape;
        for (int r = i; r < n && a.n < kMaxSegs; ++r) {
            const SpmmBwdJob& q = jobs[r];
            if ((done >> r & 1) || q.At->nnz == 0 || bwd_kind(q.k) != kind) continue;
            done |= 1ull << r;
            shape.add(q.At->n_rows, q.At->n_cols, q.At->nnz);
            SpmmBwdSeg& g = a.s[a.n++];
            g.rowptr = q.At->rowptr; g.colidx = q.At->colidx; g.avals = q.At->vals;
            g.dH = q.dH; g.xs_idx = q.xs_idx; g.dXs = q.dXs;
            g.N = (int)q.At->n_rows; g.k = q.k; g.accumulate = q.accumulate ? 1 : 0;
        }
        switch (kind) {
            case 1: launch_bwd_kernel<1, 4, false, false>(a, shape, DegreeK{}, s); break;
            case 2: launch_bwd_kernel<2, 4, false, false>(a, shape, DegreeK{}, s); break;
            case 4: launch_bwd_kernel<4, 2, false, false>(a, shape, DegreeK{}, s); break;
            default: launch_bwd_kernel<8, 1, false, false>(a, shape, DegreeK{}, s); break;
        }
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

// The dense input gradient of several kinds of source rows (k <= kDenseMaxK).
int launch_spmm_dense(const SpmmDenseJob* jobs, int n, int D, hipStream_t s, PendingSums* pending) {
    unsigned long long done = 0;
    for (int i = 0; i < n; ++i) {
        if ((done >> i & 1) || jobs[i].n_rows == 0) continue;
        const int kind = bwd_kind(jobs[i].k);
        SpmmBwdArgs a{};
        a.D = D;
        LaunchShape shape;
        for (int r = i; r < n && a.n < kMaxSegs; ++r) {
            const SpmmDenseJob& q = jobs[r];
            if ((done >> r & 1) || q.n_rows == 0 || bwd_kind(q.k) != kind) continue;
            done |= 1ull << r;
            shape.add(q.n_rows, q.At ? q.At->n_cols : 0, 0);
            SpmmBwdSeg& g = a.s[a.n++];
            if (q.At) { g.rowptr = q.At->rowptr; g.colidx = q.At->colidx; g.avals = q.At->vals; }
            if (q.At2) { g.rowptr2 = q.At2->rowptr; g.colidx2 = q.At2->colidx; g.avals2 = q.At2->vals; g.col2_off = q.col2_off; }
            g.dH = q.dH; g.xs_idx = q.idx; g.dXs = q.dX;
            g.N = (int)q.n_rows; g.k = q.k;
            g.init = q.init; g.gate = q.gate;
            g.more[0] = q.more[0]; g.more[1] = q.more[1];
        }
        bool last = true;
        for (int r = 0; r < n; ++r) last = last && ((done >> r & 1) || jobs[r].n_rows == 0);
        PendingSums sums{};
        if (last && pending) {
            sums = *pending;
            pending->n = 0;
        }
        switch (kind) {
            case 1: launch_bwd_kernel<1, 4, false, true>(a, shape, DegreeK{}, s, sums); break;
            case 2: launch_bwd_kernel<2, 4, false, true>(a, shape, DegreeK{}, s, sums); break;
            case 4: launch_bwd_kernel<4, 2, false, true>(a, shape, DegreeK{}, s, sums); break;
            default: launch_bwd_kernel<8, 1, false, true>(a, shape, DegreeK{}, s, sums); break;
        }
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_spmm_bwd(const dr_csr* At, const float* dH, const uint16_t* xs_idx, int D, int k, float* dXs,
                    int accumulate, hipStream_t s) {
    const SpmmBwdJob j{At, dH, xs_idx, k, dXs, accumulate};
    return launch_spmm_bwds(&j, 1, D, s);
}

int launch_spmm_bwd_adaptive(const dr_csr* At, const uint8_t* edge_class, const float* dH, const uint16_t* xr_idx, int D,
                             const dr_degree_classes* c, float* dXr, int accumulate, hipStream_t s) {
    if (At->nnz == 0) {
        if (accumulate) return DR_OK;
        return launch_fill_u32(reinterpret_cast<uint32_t*>(dXr), (size_t)At->n_rows * c->k1, 0u, s);
    }
    const DegreeK dk{c->t1, c->t2, c->k2, c->k3};
    SpmmBwdArgs a{};
    a.D = D;
    a.n = 1;
    LaunchShape shape;
    shape.add(At->n_rows, At->n_cols, At->nnz);
    SpmmBwdSeg& g = a.s[0];
    g.rowptr = At->rowptr; g.colidx = At->colidx; g.avals = At->vals; g.ecls = edge_class;
    g.dH = dH; g.xs_idx = xr_idx; g.dXs = dXr;
    g.N = (int)At->n_rows; g.k = c->k1; g.accumulate = accumulate ? 1 : 0;
    switch (bwd_kind(c->k1)) {
        case 1: launch_bwd_kernel<1, 4, true, false>(a, shape, dk, s); break;
        case 2: launch_bwd_kernel<2, 4, true, false>(a, shape, dk, s); break;
        case 4: launch_bwd_kernel<4, 2, true, false>(a, shape, dk, s); break;
        default: launch_bwd_kernel<8, 1, true, false>(a, shape, dk, s); break;   // k <= 64: one window of slots (checked by the caller)
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

// class (0 low, 1 medium, 2 high) of the destination of every stored entry of At, from the forward row pointers
__global__ __launch_bounds__(256) void edge_class_kernel(const int32_t* __restrict__ t_colidx, int nnz,
                                                         const int32_t* __restrict__ a_rowptr, int t1, int t2,
                                                         uint8_t* __restrict__ out) {
    for (uint32_t e = blockIdx.x * 256 + threadIdx.x; e < (uint32_t)nnz; e += gridDim.x * 256) {
        const int i = t_colidx[e];
        const int deg = a_rowptr[i + 1] - a_rowptr[i];
        out[e] = (uint8_t)(deg <= t1 ? 0 : (deg <= t2 ? 1 : 2));
    }
}

int launch_edge_classes(const dr_csr* At, const int32_t* a_rowptr, const dr_degree_classes* c, uint8_t* out, hipStream_t s) {
    if (At->nnz == 0) return DR_OK;
    unsigned blocks = (unsigned)((At->nnz + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(edge_class_kernel, dim3(blocks), dim3(256), 0, s, At->colidx, (int)At->nnz, a_rowptr, c->t1, c->t2, out);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

}  // namespace drc
