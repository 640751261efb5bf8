// Dense part of the HeteroConv layer (paper Section 3.2, matrix form Y = A X W, and its gradients in
// Section 3.3): the per-relation linear projections and the weight gradients on the matrix cores, with the
// element-wise glue fused in:
//   - the D-ReLU output enters as CBSR and is densified on the fly into the LDS operand tile;
//   - the max-merge is formed in registers from both cell branches (forward), its mask gates the upstream gradient as
//     it enters (backward);
//   - the self-term gradient is sampled at the saved CBSR indices and leaves compact.
//
// Arithmetic.  Operands are fp32, the matrix cores' fp32 rate is 155 TFLOP/s (measured from registers) and was what bound
// these kernels.  Each fp32 number is therefore written as the sum of three bf16 numbers, x = x1 + x2 + x3 (round to
// nearest each time: 3 x 8 significant bits hold all 24, so from about 2^-108 upwards the sum is exact; smaller numbers lose
// what lies below bf16's smallest, 2^-133), and a product is formed from six bf16 products, x1 y1 + x1 y2 + x2 y1 +
// x1 y3 + x2 y2 + x3 y1, each exact.  What is left out, x2 y3 + x3 y2 + x3 y3, is below 2^-25 |x y|: half an ulp of one fp32
// rounding, which an fp32 multiply-add commits for every term anyway.  The leading products x1 y1 and the five small ones
// have accumulators of their own: the small sum is added once, with one rounding, and it can be left out where the leading
// one is not finite, so that infinite and overflowing products are what they are in fp32 (with_small).
// Six bf16 products run at 250 .. 300 TFLOP/s of fp32 work.  Every operand is read once for all the products it takes part in: memory
// is then no longer what these kernels wait for, but the issue of vector and matrix instructions is (below).
//
// Layouts.  The 16x16x32 instruction takes eight consecutive contraction indices per lane, as one 16-byte register
// group.  LDS holds the operand tile in exactly those units, one plane per part.  The contraction index is permuted
// (unit u = columns 4u .. 4u+3 and D/2+4u .. D/2+4u+3) so that the global loads behind a unit are two fully coalesced
// float4 loads; the weights follow the same order.  The weights are the first operand and the activations the second, so
// a lane ends up with four consecutive output columns of one row: one 16-byte store per 16 rows.
//
// Pipeline.  Eight wavefronts per workgroup, two per SIMD, LDS tiles doubled, one barrier per tile.  In every step
// the wavefronts of the first half split and stage the next tile and then multiply the current one, those of the second half
// multiply first: on each SIMD the vector instructions of one wavefront run under the matrix instructions of the other.
// (With both halves in step and one LDS buffer a 1.2 M-row forward took 0.72 ms.)
//
// What a tile costs (32 cells, D = 128; parts switched off one by one): staging alone and multiplying alone take about as long
// as one another, and together little less than their sum.  A matrix instruction takes 16 clocks of the SIMD and keeps vector
// instructions out for 8 of them; LDS reads come at 256 bytes a clock, writes at 80.  Forward projection of 250 000 cells and
// 180 000 nets: 204 -> 191 us with fragments read ahead, conflict-free places in LDS and graph descriptors in registers;
// global memory is no longer what it waits for (without any loads and stores 188).  Vector and matrix instructions of a SIMD's two
// wavefronts take turns for the most part: 202 -> 192 (a launch each) with 382 -> 296 vector instructions per wavefront and tile of cells (the scattered
// operand in units of eight neighbouring columns, cleared without a loop) and matrix instructions issued first.  Not kept: blocks of
// 256 rows whose operands stay in registers while the weights pass by in LDS (1.2 M cells 660 -> 758: a barrier every 16 columns, and
// more splitting in all); wavefronts with 32 columns and
// all registers of a SIMD (241), and staging spread between the matrix instructions of the same wavefront (201).
#include "dr_internal.h"
#include "wgrad_shape.h"

#include <type_traits>

namespace drc {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Keeps `base + constant` in that form: the compiler would merge the constant into known-zero bits of the base and then
// no longer find it for the instruction's own offset field.  Inside a loop: what is computed from it is computed there and
// does not hold a register over the multiply.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

template <int D> struct Tile {
    static constexpr int NB = D / 16;                              // 16-column blocks = wavefronts side by side
    static constexpr int WAVES = D == 96 ? 6 : 8;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int RG = WAVES / NB;                          // row groups of 32 rows (wavefronts one below the other)
    static constexpr int BM = 32 * RG;                             // rows per tile
    static constexpr int KU = D / 8;                               // 16-byte units per row and part
    static constexpr int KS = D / 32;                              // MFMA steps
    static constexpr int TPR = D == 128 ? 16 : (D == 32 ? 4 : 8);  // threads that share one CBSR row; a row never straddles wavefronts
    static constexpr int PLANE = KU * BM + KU / 2;                 // units per part (unit_at)
    static constexpr int OPER = 3 * PLANE;                         // units per operand
    static_assert(BM * KU == THREADS && BM * TPR <= THREADS && 64 % TPR == 0, "one unit per thread");
};

// Place of a unit in its plane.  A 16-byte LDS read is served in groups of 16 lanes that mix the rows of two neighbouring
// units: lanes 0-3, 12-15 and 20-27 of the first 32, and the rest (measured pair by pair), so those two units have to start
// on the same bank; the pairs 2h, 2h + 1 of one row start 16 bytes further on each.  (A gap after every unit made every read of a
// fragment a two-way conflict.)
template <int D> __device__ __forceinline__ int unit_at(int unit, int row) { return unit * Tile<D>::BM + (unit >> 1) + row; }
// The unit that thread t of a row stages.  At D = 128 neighbouring threads take units of different pairs, so that eight of them write
// to eight different banks: dproj of 250 000 cells and 180 000 nets 131 -> 128 and 73 -> 70 us, forward 131 -> 130.  (Narrower rows
// have fewer than eight pairs; at D = 96 the forward became 1 % slower.)
template <int D> __device__ __forceinline__ int unit_of(int t) {
    constexpr int H = Tile<D>::KU / 2;
    return D == 128 ? (t < H ? 2 * t : 2 * (t - H) + 1) : t;
}

// Three bf16 parts of half of each of eight numbers, two at a time (one conversion instruction makes two parts).
// Half, so that no finite number rounds up to an infinite first part; kUnscale takes a sum of products back.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr float kScale = 0.5f;
static_assert(kScale * kScale * kUnscale == 1.0f);
struct Split8 { bf16x8 p[3]; };
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ float low_part(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float high_part(uint32_t v) { return __builtin_bit_cast(float, v & 0xffff0000u); }
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
    uint32_t w[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = kScale * x[2 * j], b = kScale * x[2 * j + 1];
        w[0][j] = pack2(a, b);
        const float ra = a - low_part(w[0][j]), rb = b - high_part(w[0][j]);
        w[1][j] = pack2(ra, rb);
        w[2][j] = pack2(ra - low_part(w[1][j]), rb - high_part(w[1][j]));
    }
    Split8 s;
#pragma unroll
    for (int p = 0; p < 3; ++p) s.p[p] = __builtin_bit_cast(bf16x8, w[p]);
    return s;
}
// the parts of `s` where keep(j) holds, zero elsewhere
template <typename K> __device__ __forceinline__ Split8 select8(const Split8& s, K keep) {
    uint32_t m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) m[j] = (keep(2 * j) ? 0x0000ffffu : 0u) | (keep(2 * j + 1) ? 0xffff0000u : 0u);
    Split8 r;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        struct Words { uint32_t w[4]; } v = __builtin_bit_cast(Words, s.p[p]);
#pragma unroll
        for (int j = 0; j < 4; ++j) v.w[j] &= m[j];
        r.p[p] = __builtin_bit_cast(bf16x8, v);
    }
    return r;
}
// the three parts of (half of) one number, `stride` bf16 numbers apart
__device__ __forceinline__ void put_parts(__bf16* at, int stride, float v) {
    v *= kScale;
    const __bf16 a = (__bf16)v;
    const float r = v - (float)a;
    const __bf16 b = (__bf16)r;
    at[0] = a;
    at[stride] = b;
    at[2 * stride] = (__bf16)(r - (float)b);
}

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// hi: sum of the leading products, lo: of the five small ones
struct Acc { f32x4 hi, lo; };
// The sum of leading products and small ones.  An infinite or overflowing operand makes the leading sum infinite or
// not-a-number as in fp32, but its remainder is not-a-number and its small products may be infinities of either sign: the
// small sum must not decide then, and it is finite whenever the leading one is.
constexpr float kFloatMax = 3.4028234663852886e38f;
__device__ __forceinline__ f32x4 with_small(const f32x4& hi, const f32x4& lo, float m = kFloatMax) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = hi[r] + __builtin_amdgcn_fmed3f(lo[r], -m, m);     // (not-a-number: -m)
    return v;
}
__device__ __forceinline__ f32x4 total(const Acc& c) {
    return kUnscale * with_small(c.hi, c.lo, __builtin_bit_cast(float, opaque(__builtin_bit_cast(int, kFloatMax))));
}
// Row blocks are read and written through buffer descriptors: the base is the block's first row and the size ends with
// the array, so rows past the end read as zero and are not written.  No access in the pipelines is conditional, which
// lets the compiler count exactly how many may still be outstanding (a store under a branch makes every later wait for a
// load wait for the store as well), and the rows of a block need one offset register.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
using Buf = __amdgpu_buffer_rsrc_t;
constexpr int kNt = 2;                    // cache policy: streamed
constexpr int kNowhere = 0x7ffffff0;      // an offset outside every block
// (a descriptor has to be uniform for the compiler too, and parts of this address arithmetic may be done per lane)
__device__ __forceinline__ Buf block_view(const void* p, int rows_left, int row_bytes) {
    const int rows = __builtin_amdgcn_readfirstlane(min(max(rows_left, 0), 1 << 16));
    const uint64_t at = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)hi << 32 | lo), (short)0, rows * row_bytes, 0x00020000);
}
__device__ __forceinline__ f32x4 load4(Buf b, int off) { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, kNt)); }
__device__ __forceinline__ float load1(Buf b, int off) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, kNt)); }
__device__ __forceinline__ uint32_t load1u(Buf b, int off) { return __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, kNt); }
template <int CP = 0> __device__ __forceinline__ void store4(Buf b, int off, const f32x4& v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, off, 0, CP);
}

// The two halves of a workgroup's wavefronts run loops of their own (yes: stage, then multiply).  With one loop and the
// staging under `if (half)` the compiler has to assume that a wavefront may change sides from one trip to the next: the
// waits in front of the staging and of the multiply then covered loads and stores that had only just been issued, and every
// trip stood for a whole memory latency.
template <int N, int I = 0, typename F> __device__ __forceinline__ void steps(F f) {       // f(0), ..., f(N - 1), each a constant
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        steps<N, I + 1>(f);
    }
}
struct yes { static constexpr bool value = true; };
struct no { static constexpr bool value = false; };
// Stores that write nothing, behind the first prefetch of a loop in which stores come behind the prefetch: the number of
// operations that may be outstanding at the loop's first wait is the smaller one of the way in and of the way round.
template <int N> __device__ __forceinline__ void pad_stores(float* p) {
    const Buf b = block_view(p, 0, 0);
#pragma unroll
    for (int i = 0; i < N; ++i) __builtin_amdgcn_raw_buffer_store_b32(0u, b, kNowhere - 4 * i, 0, 0);
}

// Weight fragments of one 16-column block: output column n = first + (lane & 15), unit 4 s + (lane >> 4) per step.
// TRANS: B[k][n] = W[n][k].  PLAIN: unit u = columns 8u .. 8u+7 (the scattered operand).
template <int D, bool TRANS, bool PLAIN = false>
__device__ __forceinline__ void load_weight(const float* __restrict__ W, int first, int lane, bf16x8 (&w)[Tile<D>::KS][3]) {
    const int n = first + (lane & 15);
#pragma unroll
    for (int s = 0; s < Tile<D>::KS; ++s) {
        const int u = 4 * s + (lane >> 4);
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = PLAIN ? 8 * u + j : 4 * u + (j & 3) + (j >> 2) * (D / 2);
            x[j] = TRANS ? W[(size_t)n * D + k] : W[(size_t)k * D + n];
        }
        const Split8 sp = split8(x);
#pragma unroll
        for (int p = 0; p < 3; ++p) w[s][p] = sp.p[p];
    }
}

// A kernel's arguments, read where they lie: loads from the constant address space are scalar whatever is stored in
// between, so that descriptors built from them are uniform.
#define DRC_CONST __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ const DRC_CONST T* kernel_args() {
    return (const DRC_CONST T*)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
}

// The graph whose tiles hold tile `t` (tile0 of the graphs is increasing; t only grows).  Its descriptor is kept in scalar
// registers and fetched when the graph changes: read anew for every tile, the chain of scalar loads, each waited for together
// with all LDS traffic in flight, took longer than the arithmetic of the staging.
template <typename SEG> struct Place {
    SEG g;
    int q, end;                   // graph, and the first tile past it
    __device__ __forceinline__ void start(const DRC_CONST SEG* s, int n, int t) {
        q = 0;
        end = n > 1 ? s[1].tile0 : 0x7fffffff;
        g = fetch(s);
        seek(s, n, t);
    }
    __device__ __forceinline__ void seek(const DRC_CONST SEG* s, int n, int t) {
        if (t < end) return;
        do {
            ++q;
            end = q + 1 < n ? s[q + 1].tile0 : 0x7fffffff;
        } while (t >= end);
        g = fetch(s + q);
    }
};

// CBSR rows -> operand tile.  Pairs ppart, ppart + TPR, ... of a row belong to thread (row, ppart); the first kPairs per
// thread travel through registers, further ones (wide selections) are fetched when they are placed.
constexpr int kPairs = 4;
struct PairRegs { float v[kPairs]; uint32_t c[kPairs]; };

// pairs of row `row` of a block whose selections start at `vals`, `idx`
template <int TPR>
__device__ __forceinline__ void load_pairs(PairRegs& r, Buf vals, Buf idx, int k, int row, int ppart) {
    const int at4 = opaque((row * k + ppart) * 4), at2 = opaque((row * k + ppart) * 2);
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
        r.v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vals, at4 + TPR * u * 4, 0, 0));
        r.c[u] = __builtin_amdgcn_raw_buffer_load_b16(idx, at2 + TPR * u * 2, 0, 0);
    }
}

// `on` false: goes to the gap behind the last unit
template <int D> __device__ __forceinline__ void put_pair(bf16x8* plane, bool on, int row, int col, float v) {
    using T = Tile<D>;
    const int at = on ? unit_at<D>(col >> 3, row) * 8 + (col & 7) : (T::PLANE - 1) * 8;
    put_parts(reinterpret_cast<__bf16*>(plane) + at, 8 * T::PLANE, v);
}

// rows past the end hold zeros at column 0
template <int D>
__device__ __forceinline__ void stage_cbsr(bf16x8* oper, const PairRegs& pr, const float* __restrict__ vals,
                                           const uint16_t* __restrict__ idx, int k, int rows_left, int row, int ppart) {
    using T = Tile<D>;
    ppart = opaque(ppart);
    const int none = opaque(0);
    struct Words { int w[4]; };
    const bf16x8 z = __builtin_bit_cast(bf16x8, Words{none, none, none, none});
#pragma unroll
    for (int u = 0; u < T::KU; u += T::TPR)
        if (T::KU % T::TPR == 0 || u + ppart < T::KU) {
#pragma unroll
            for (int p = 0; p < 3; ++p) oper[p * T::PLANE + unit_at<D>(u + ppart, row)] = z;
        }
    // the threads of a row sit in one wavefront and LDS executes a wavefront's accesses in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int u = 0; u < kPairs; ++u)
            put_pair<D>(oper, ppart + T::TPR * u < k, row, (int)pr.c[u], pr.v[u]);
    if (k > T::TPR * kPairs && row < rows_left)
        for (int t = ppart + T::TPR * kPairs; t < k; t += T::TPR) put_pair<D>(oper, true, row, idx[(size_t)row * k + t], vals[(size_t)row * k + t]);
}

// dense unit -> operand tile
template <int D> __device__ __forceinline__ void stage_unit(bf16x8* oper, int row, int unit, const Split8& s) {
    using T = Tile<D>;
#pragma unroll
    for (int p = 0; p < 3; ++p) oper[p * T::PLANE + unit_at<D>(unit, row)] = s.p[p];
}

// The activations' fragments of one step (32 rows, one contraction block): a part's registers are read again for the next step
// as soon as its last product is issued, and the leading part, which is used last, may have two sets (SETS), so that LDS
// latency passes under matrix instructions.  (Whole second sets would not fit the registers beside the weights.)
template <int SETS> struct Frags { bf16x8 p0[SETS][2], p1[2], p2[2]; };
template <int D> __device__ __forceinline__ void load_part(const bf16x8* oper, int part, int s, int rg, int lane, bf16x8 (&x)[2]) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
        x[rb] = oper[part * Tile<D>::PLANE + unit_at<D>(4 * s + (lane >> 4), rg * 32 + rb * 16 + (lane & 15))];
}
// Step STEP's products with NW weights: w[i] the parts of a weight's fragment, c[i] its accumulators for two tiles of rows.
// MORE: a step follows, whose fragments are at (next, s).  Consecutive instructions go to different accumulators.  The small
// products are added in the order in which that frees the fragments, x3 y1, x2 y2, x2 y1, x1 y3, x1 y2: one of about 2^-16 comes after
// one of 2^-8, which costs less than half an ulp of the small sum, 2^-32 of the whole.
template <int D, int STEP, bool MORE, int NW, int SETS>
__device__ __forceinline__ void multiply(const bf16x8* const (&w)[NW], Acc (*const (&c)[NW])[2], Frags<SETS>& x, const bf16x8* next, int s,
                                         int rg, int lane) {
    constexpr int set = STEP % SETS;
    if constexpr (MORE && SETS == 2) load_part<D>(next, 0, s, rg, lane, x.p0[set ^ 1]);
    __builtin_amdgcn_sched_barrier(0);
    const auto small = [&](int part, const bf16x8 (&f)[2]) {
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) (*c[i])[rb].lo = mfma(w[i][part], f[rb], (*c[i])[rb].lo);
    };
    small(0, x.p2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MORE) load_part<D>(next, 2, s, rg, lane, x.p2);
    __builtin_amdgcn_sched_barrier(0);
    small(1, x.p1);
    small(0, x.p1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MORE) load_part<D>(next, 1, s, rg, lane, x.p1);
    __builtin_amdgcn_sched_barrier(0);
    small(2, x.p0[set]);
    small(1, x.p0[set]);
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) (*c[i])[rb].hi = mfma(w[i][0], x.p0[set][rb], (*c[i])[rb].hi);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MORE && SETS == 1) load_part<D>(next, 0, s, rg, lane, x.p0[0]);
}
// The same without reading ahead, the small products smallest first; the compiler places the reads.
template <int D, int NW>
__device__ __forceinline__ void multiply_now(const bf16x8* const (&w)[NW], Acc (*const (&c)[NW])[2], const bf16x8* oper, int s, int rg, int lane) {
    bf16x8 x[3][2];
#pragma unroll
    for (int p = 0; p < 3; ++p) load_part<D>(oper, p, s, rg, lane, x[p]);
    constexpr int W[5] = {2, 0, 1, 1, 0}, X[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
#pragma unroll
        for (int j = 0; j < 5; ++j)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) (*c[i])[rb].lo = mfma(w[i][W[j]], x[X[j]][rb], (*c[i])[rb].lo);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) (*c[i])[rb].hi = mfma(w[i][0], x[0][rb], (*c[i])[rb].hi);
    }
}
template <int D, int SETS> __device__ __forceinline__ void first_frags(const bf16x8* oper, int rg, int lane, Frags<SETS>& x) {
    load_part<D>(oper, 2, 0, rg, lane, x.p2);
    load_part<D>(oper, 1, 0, rg, lane, x.p1);
    load_part<D>(oper, 0, 0, rg, lane, x.p0[0]);
}

// ---------------------------------------------------------------------------------------------------
// forward:  cells  Y = max(Xs W_self + H_near W_neigh, H_pinned W_pinned), mask      (three weights)
//           nets   Y = Xs W_self + H_pins W_neigh                                     (two weights)
// A workgroup keeps the weights of its side in registers (wavefront w: 16 output columns, 48 registers per weight at
// D = 128) and walks over row tiles of that side; the loads of the next tile are in flight during the multiply.  One read of
// every operand, one write of Y: separate kernels for near and for pinned + merge wrote Y twice and read it once in
// between.
// ---------------------------------------------------------------------------------------------------
struct ProjFwdSide {              // one graph's rows of one node type
    const float *vals, *H1, *H2;  // CBSR of the self term, H_near / H_pins, H_pinned (cells)
    const uint16_t* idx;
    float* Y;
    uint8_t* mask;
    int rows, k, tile0;
};
__device__ __forceinline__ ProjFwdSide fetch(const DRC_CONST ProjFwdSide* s) {
    return ProjFwdSide{s->vals, s->H1, s->H2, s->idx, s->Y, s->mask, s->rows, s->k, s->tile0};
}
struct ProjFwdArgs {
    ProjFwdSide cell[kMaxGraphs], net[kMaxGraphs];
    const float *w_self_near, *w_neigh_near, *w_pinned, *w_self_pins, *w_neigh_pins;
    int n, cell_tiles, net_tiles, cell_wgs, relu;
};
static_assert(sizeof(ProjFwdArgs) < 4096, "kernel arguments");

// CP: cache policy of the stores.  A wavefront writes 64 bytes of a row of Y and 16 of the mask, others the rest of a line.
// Through the L2 the pieces leave as one line; streamed, they leave one by one (1.2 M x 128 cells: 1.53 GB counted as written
// for the 0.77 GB that leave through the L2).  What the L2 still holds at the end is written back before the next launch may start, so the stores are
// streamed while all of Y would stay there (kL2Bytes, eight of 4 MB).  Through the L2 / streamed: layer of 1.2 M cells, D = 128
// 6.14 / 6.22 ms, 250 000 cells 1.234 / 1.245, 60 000 cells, D = 64 0.206 / 0.203, 33 331 cells, D = 96 0.239 / 0.235.
constexpr int64_t kL2Bytes = 32ll << 20;
template <int D, bool CELL, int CP>
__device__ __forceinline__ void proj_fwd_side(const DRC_CONST ProjFwdArgs* a, bf16x8* smem, int wg, int n_wg) {
    using T = Tile<D>;
    const DRC_CONST ProjFwdSide* const segs = CELL ? a->cell : a->net;
    const int tiles = CELL ? a->cell_tiles : a->net_tiles, n = a->n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = wave % T::NB, rg = wave / T::NB;
    const bool relu = a->relu != 0;
    const int urow = tid / T::KU, unit = unit_of<D>(tid % T::KU);              // this thread's unit of a dense operand
    const int prow = tid / T::TPR, ppart = tid % T::TPR;           // past the tile (D = 96): reads nothing, writes nothing
    const bool pairs = wave * 64 < T::BM * T::TPR;                 // whole wavefronts

    bf16x8 wS[T::KS][3], w1[T::KS][3], w2[T::KS][3];
    load_weight<D, false, true>(CELL ? a->w_self_near : a->w_self_pins, 16 * nb, lane, wS);
    load_weight<D, false>(CELL ? a->w_neigh_near : a->w_neigh_pins, 16 * nb, lane, w1);
    if constexpr (CELL) load_weight<D, false>(a->w_pinned, 16 * nb, lane, w2);

    f32x4 h1[2], h2[2];
    PairRegs pr;
    const int uoff = opaque((urow * D + 4 * unit) * 4);                    // bytes from the first row of the tile
    auto prefetch = [&](const ProjFwdSide& g, int t) {             // past the last tile: reads nothing
        const int base = (t - g.tile0) * T::BM, left = t < tiles ? g.rows - base : 0;
        const Buf b1 = block_view(g.H1 + (size_t)base * D, left, D * 4);
        h1[0] = load4(b1, uoff);
        h1[1] = load4(b1, uoff + D * 2);
        if constexpr (CELL) {
            const Buf b2 = block_view(g.H2 + (size_t)base * D, left, D * 4);
            h2[0] = load4(b2, uoff);
            h2[1] = load4(b2, uoff + D * 2);
        }
        load_pairs<T::TPR>(pr, block_view(g.vals + (size_t)base * g.k, left, g.k * 4), block_view(g.idx + (size_t)base * g.k, left, g.k * 2),
                           g.k, prow, ppart);
    };
    auto commit = [&](const ProjFwdSide& g, int t, bf16x8* buf) {
        const int base = (t - g.tile0) * T::BM;
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = h1[j >> 2][j & 3];
        stage_unit<D>(buf + T::OPER, urow, unit, split8(x));
        if constexpr (CELL) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = h2[j >> 2][j & 3];
            stage_unit<D>(buf + 2 * T::OPER, urow, unit, split8(x));
        }
        if (pairs) stage_cbsr<D>(buf, pr, g.vals + (size_t)base * g.k, g.idx + (size_t)base * g.k, g.k, t < tiles ? g.rows - base : 0, prow, ppart);
    };
    if (wg >= tiles) return;
    const auto walk = [&](auto first) {
        constexpr bool kFirst = decltype(first)::value;
        int t = wg;
        Place<ProjFwdSide> here, ahead;           // of tile t; of the next one, and in the loop of the one after
        here.start(segs, n, t);
        prefetch(here.g, t);
        commit(here.g, t, smem);
        ahead = here;
        ahead.seek(segs, n, t + n_wg);
        prefetch(ahead.g, t + n_wg);
        if constexpr (kFirst) pad_stores<CELL ? 4 : 2>(here.g.Y);          // a tile's stores come behind its prefetch
        __syncthreads();
        for (int cur = 0;; cur ^= 1) {
            const ProjFwdSide g = here.g, g1 = ahead.g;
            const int base = (t - g.tile0) * T::BM, t1 = t + n_wg;
            bf16x8* const buf = smem + cur * 3 * T::OPER;
            here = ahead;
            ahead.seek(segs, n, t1 + n_wg);
            auto stage_next = [&]() {
                __builtin_amdgcn_s_setprio(0);
                commit(g1, t1, smem + (cur ^ 1) * 3 * T::OPER);
                prefetch(ahead.g, t1 + n_wg);
                __builtin_amdgcn_s_setprio(1);
            };
            if constexpr (kFirst) stage_next();
            __builtin_amdgcn_sched_barrier(0);
            // One operand after the other, so that the accumulators of near are down to its values when pinned begins: the
            // registers then hold the fragments of the next step too, whose LDS reads run under this step's products.
            Acc c[2] = {};
            f32x4 near[2];
            Frags<2> x;
            constexpr int NS = (CELL ? 3 : 2) * T::KS;
            first_frags<D>(buf, rg, lane, x);
            steps<NS>([&](auto step) {
                constexpr int i = decltype(step)::value, s = i % T::KS, o = i / T::KS;
                const bf16x8* const next = buf + (i + 1) / T::KS * T::OPER;
                const bf16x8* const w[1] = {o == 0 ? wS[s] : (o == 1 ? w1[s] : w2[s])};
                Acc(*const acc[1])[2] = {&c};
                multiply<D, i, i + 1 < NS>(w, acc, x, next, (i + 1) % T::KS, rg, lane);
                if constexpr (CELL && i == 2 * T::KS - 1) {
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) {
                        near[rb] = total(c[rb]);
                        c[rb] = Acc{};
                    }
                }
            });
            const Buf by = block_view(g.Y + (size_t)base * D, g.rows - base, D * 4);
            const Buf bm = block_view(g.mask + (size_t)base * D, g.rows - base, D);
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                const int ln = opaque(lane), at = (rg * 32 + rb * 16 + (ln & 15)) * D + 16 * nb + 4 * (ln >> 4);
                f32x4 v = total(c[rb]);
                if constexpr (CELL) {             // mask = [near >= pinned]
                    const f32x4 p = v;
                    v = near[rb];
                    uint32_t m = 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool near_wins = v[r] >= p[r];
                        m |= near_wins ? 1u << (8 * r) : 0u;
                        v[r] = near_wins ? v[r] : p[r];
                    }
                    __builtin_amdgcn_raw_buffer_store_b32(m, bm, at, 0, CP);
                }
                if (relu) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
                }
                store4<CP>(by, at * 4, v);
            }
            if constexpr (!kFirst) stage_next();
            if (t1 >= tiles) break;
            __syncthreads();
            t = t1;
        }
    };
    if (wave < T::WAVES / 2) walk(yes{});
    else walk(no{});
}

template <int D, int CP>
__global__ __launch_bounds__(Tile<D>::THREADS, 2) void proj_kernel(ProjFwdArgs a) {
    extern __shared__ bf16x8 smem8[];
    const DRC_CONST ProjFwdArgs* const k = kernel_args<ProjFwdArgs>();
    if ((int)blockIdx.x < k->cell_wgs) proj_fwd_side<D, true, CP>(k, smem8, blockIdx.x, k->cell_wgs);
    else proj_fwd_side<D, false, CP>(k, smem8, blockIdx.x - k->cell_wgs, gridDim.x - k->cell_wgs);
}

// ---------------------------------------------------------------------------------------------------
// backward:  cells  dZ_near = dY where mask == 1, dZ_pinned = dY where mask == 0
//                   dH_near = dZ_near W_neigh^T,  dH_pinned = dZ_pinned W_pinned^T,
//                   S[row, t] = (dZ_near W_self^T)[row, idx[row, t]]
//            nets   dH_pins = dY W_neigh^T,  S[row, t] = (dY W_self^T)[row, idx[row, t]]
// dY and the mask are read once for all three products; the self term leaves compact ([rows, k]), so that the kernel that
// sums the transposed relations can add it and write the dense dX (it used to read dY and the mask again, in a kernel of
// its own).
// ---------------------------------------------------------------------------------------------------
struct ProjBwdSide {
    const float* dY;
    const uint8_t* mask;          // cells
    float *dH1, *dH2;             // dH_near / dH_pins, dH_pinned (cells)
    const uint16_t* idx;
    float* S;
    int rows, k, tile0;
};
__device__ __forceinline__ ProjBwdSide fetch(const DRC_CONST ProjBwdSide* s) {
    return ProjBwdSide{s->dY, s->mask, s->dH1, s->dH2, s->idx, s->S, s->rows, s->k, s->tile0};
}
template <int G> struct ProjBwdArgs {         // of up to G graphs
    ProjBwdSide cell[G], net[G];
    const float *w_self_near, *w_neigh_near, *w_pinned, *w_self_pins, *w_neigh_pins;
    int n, cell_tiles, net_tiles, cell_wgs, net_wgs;
};
static_assert(sizeof(ProjBwdArgs<kMaxGraphs>) < 4096, "kernel arguments");

template <int D, bool CELL, typename ARGS>
__device__ __forceinline__ void proj_bwd_side(const DRC_CONST ARGS* a, bf16x8* smem, int wg, int n_wg) {
    using T = Tile<D>;
    constexpr int LDC = D + 4;
    const DRC_CONST ProjBwdSide* const segs = CELL ? a->cell : a->net;
    const int tiles = CELL ? a->cell_tiles : a->net_tiles, n = a->n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = wave % T::NB, rg = wave / T::NB;
    const int urow = tid / T::KU, unit = unit_of<D>(tid % T::KU);
    const int prow = tid / T::TPR, ppart = tid % T::TPR;           // past the tile (D = 96): reads nothing, writes nothing
    float* const sC0 = reinterpret_cast<float*>(smem + 4 * T::OPER);          // [2][BM][LDC] self-term products

    bf16x8 wS[T::KS][3], w1[T::KS][3], w2[T::KS][3];
    load_weight<D, true>(CELL ? a->w_self_near : a->w_self_pins, 16 * nb, lane, wS);
    load_weight<D, true>(CELL ? a->w_neigh_near : a->w_neigh_pins, 16 * nb, lane, w1);
    if constexpr (CELL) load_weight<D, true>(a->w_pinned, 16 * nb, lane, w2);

    f32x4 y[2];
    uint32_t mk[2];
    const int uoff = opaque((urow * D + 4 * unit) * 4), moff = opaque(urow * D + 4 * unit);   // from the first row of the tile
    auto prefetch = [&](const ProjBwdSide& g, int t) {             // past the last tile: reads nothing
        const int base = (t - g.tile0) * T::BM, left = t < tiles ? g.rows - base : 0;
        const Buf by = block_view(g.dY + (size_t)base * D, left, D * 4);
        y[0] = load4(by, uoff);
        y[1] = load4(by, uoff + D * 2);
        if constexpr (CELL) {
            const Buf bm = block_view(g.mask + (size_t)base * D, left, D);
            mk[0] = load1u(bm, moff);
            mk[1] = load1u(bm, moff + D / 2);
        }
    };
    auto commit = [&](bf16x8* buf) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = y[j >> 2][j & 3];
        const Split8 sp = split8(x);
        if constexpr (CELL) {
            auto byte = [&](int j) { return (mk[j >> 2] >> (8 * (j & 3))) & 0xffu; };
            const Split8 s1 = select8(sp, [&](int j) { return byte(j) == 1u; }), s2 = select8(sp, [&](int j) { return byte(j) == 0u; });
            stage_unit<D>(buf, urow, unit, s1);
            stage_unit<D>(buf + T::OPER, urow, unit, s2);
        } else {
            stage_unit<D>(buf, urow, unit, sp);
        }
    };
    if (wg >= tiles) return;
    // The self-term product of a tile is sampled one step later, when all wavefronts have written theirs.
    auto sample = [&](const ProjBwdSide& g, int t, int left, const float* sC) {
        const int base = (t - g.tile0) * T::BM, at = opaque(prow) * g.k + ppart;
        left = min(left, T::BM);                  // threads past the tile (D = 96) must not reach the next tile's rows
        const Buf bi = block_view(g.idx + (size_t)base * g.k, left, g.k * 2);
        const Buf bs = block_view(g.S + (size_t)base * g.k, left, g.k * 4);
        // as loaded: a conversion here would wait for the loads before the multiply
        struct { uint16_t v[kPairs]; } col;
#pragma unroll
        for (int u = 0; u < kPairs; ++u) col.v[u] = __builtin_amdgcn_raw_buffer_load_b16(bi, (at + T::TPR * u) * 2, 0, 0);
        return [=]() {
            const int row = min(opaque(prow), T::BM - 1);
#pragma unroll
            for (int u = 0; u < kPairs; ++u) {
                uint16_t c = col.v[u];
                asm volatile("" : "+v"(c));
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sC[row * LDC + c]), bs,
                                                      ppart + T::TPR * u < g.k ? (at + T::TPR * u) * 4 : kNowhere, 0, 0);
            }
            if (g.k > T::TPR * kPairs && prow < min(left, T::BM))
                for (int p = ppart + T::TPR * kPairs; p < g.k; p += T::TPR)
                    g.S[(size_t)(base + prow) * g.k + p] = sC[prow * LDC + g.idx[(size_t)(base + prow) * g.k + p]];
        };
    };
    const auto walk = [&](auto first) {
        constexpr bool kFirst = decltype(first)::value;
        int t = wg, t0 = t;
        Place<ProjBwdSide> here, ahead;           // of tile t; of the next one, and in the loop of the one after
        here.start(segs, n, t);
        ProjBwdSide g0 = here.g;                  // of the tile before
        prefetch(here.g, t);
        commit(smem);
        ahead = here;
        ahead.seek(segs, n, t + n_wg);
        prefetch(ahead.g, t + n_wg);
        if constexpr (kFirst) pad_stores<(CELL ? 4 : 2) + kPairs>(here.g.dH1);       // a tile's stores come behind its prefetch
        __syncthreads();
        int cur = 0;
        bool have_t0 = false;
        for (;; cur ^= 1) {
            const ProjBwdSide g = here.g;
            const int base = (t - g.tile0) * T::BM, t1 = t + n_wg;
            bf16x8* const buf = smem + cur * 2 * T::OPER;
            float* const sC = sC0 + cur * T::BM * LDC;
            here = ahead;
            ahead.seek(segs, n, t1 + n_wg);
            const auto finish_t0 = sample(g0, t0, have_t0 ? g0.rows - (t0 - g0.tile0) * T::BM : 0, sC0 + (cur ^ 1) * T::BM * LDC);
            auto stage_next = [&]() {
                commit(smem + (cur ^ 1) * 2 * T::OPER);
                prefetch(ahead.g, t1 + n_wg);
            };
            if constexpr (kFirst) stage_next();
            __builtin_amdgcn_sched_barrier(0);
            // near (or the net's only branch) first, then pinned: the accumulators of both would not fit the registers
            const int ln = opaque(lane), r0 = rg * 32 + (ln & 15), c0 = 16 * nb + 4 * (ln >> 4);
            Acc c[2] = {}, cS[2] = {};
            Acc(*const both[2])[2] = {&c, &cS};
            Acc(*const one[1])[2] = {&c};
            const auto near_done = [&]() {
                const Buf b1 = block_view(g.dH1 + (size_t)base * D, g.rows - base, D * 4);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    *reinterpret_cast<f32x4*>(sC + (r0 + rb * 16) * LDC + c0) = total(cS[rb]);
                    store4(b1, ((r0 + rb * 16) * D + c0) * 4, total(c[rb]));       // gathered next: these stay in the caches
                    c[rb] = Acc{};
                }
            };
            // Fragments are read ahead where that gains: cells of D = 96 (1.2 M: 449 us, without 455) and, as much as nothing, below.  Beside
            // the weights of D = 128 they leave the compiler no registers to move reads in, and nets have one product per fragment
            // less to wait under (backward passes alone, with / without: 1.2 M cells and 0.9 M nets of D = 128 627 / 596 and 317 / 306 us,
            // nets of D = 96 236 / 230).
            if constexpr (CELL && D < 128) {
                Frags<1> x;
                constexpr int NS = 2 * T::KS;
                first_frags<D>(buf, rg, lane, x);
                steps<NS>([&](auto step) {
                    constexpr int i = decltype(step)::value, s = i % T::KS;
                    const bf16x8* const next = buf + (i + 1) / T::KS * T::OPER;
                    if constexpr (i < T::KS) {
                        const bf16x8* const w[2] = {w1[s], wS[s]};
                        multiply<D, i, i + 1 < NS>(w, both, x, next, (i + 1) % T::KS, rg, lane);
                    } else {
                        const bf16x8* const w[1] = {w2[s]};
                        multiply<D, i, i + 1 < NS>(w, one, x, next, (i + 1) % T::KS, rg, lane);
                    }
                    if constexpr (i == T::KS - 1) near_done();
                });
            } else {
#pragma unroll
                for (int s = 0; s < T::KS; ++s) {
                    const bf16x8* const w[2] = {w1[s], wS[s]};
                    multiply_now<D>(w, both, buf, s, rg, lane);
                }
                __builtin_amdgcn_sched_barrier(0);
                near_done();
                if constexpr (CELL) {
#pragma unroll
                    for (int s = 0; s < T::KS; ++s) {
                        const bf16x8* const w[1] = {w2[s]};
                        multiply_now<D>(w, one, buf + T::OPER, s, rg, lane);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (CELL) {
                const Buf b2 = block_view(g.dH2 + (size_t)base * D, g.rows - base, D * 4);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) store4(b2, ((r0 + rb * 16) * D + c0) * 4, total(c[rb]));
            }
            finish_t0();
            if constexpr (!kFirst) stage_next();
            __syncthreads();                      // this self-term tile and the next operand tiles are complete
            t0 = t;
            g0 = g;
            have_t0 = true;
            if (t1 >= tiles) break;
            t = t1;
        }
        sample(g0, t0, g0.rows - (t0 - g0.tile0) * T::BM, sC0 + cur * T::BM * LDC)();
    };
    if (wave < T::WAVES / 2) walk(yes{});
    else walk(no{});
}

template <int D>
__global__ __launch_bounds__(Tile<D>::THREADS, 2) void dproj_kernel(ProjBwdArgs<kMaxGraphs> a) {
    extern __shared__ bf16x8 smem8[];
    const DRC_CONST ProjBwdArgs<kMaxGraphs>* const k = kernel_args<ProjBwdArgs<kMaxGraphs>>();
    if ((int)blockIdx.x < k->cell_wgs) proj_bwd_side<D, true>(k, smem8, blockIdx.x, k->cell_wgs);
    else proj_bwd_side<D, false>(k, smem8, blockIdx.x - k->cell_wgs, k->net_wgs);
}

// ---------------------------------------------------------------------------------------------------
// weight gradients  dW[D,D] = A^T B, reduced over the graph's rows
//   cells  dW_neigh_near = H_near^T dZ_near,  dW_self_near = Xs^T dZ_near,  dW_pinned = H_pinned^T dZ_pinned
//   nets   dW_neigh_pins = H_pins^T dY,       dW_self_pins = Xs^T dY
// A workgroup takes every n-th chunk of rows of one side of one graph; all products of the side are accumulated in
// registers (wavefront w: 16 rows of every dW, 96 registers for three products at D = 128) from one read of every
// operand.  The contraction runs over rows, so a unit is eight rows of one column: a thread loads eight dwords down its
// column.  A wavefront is alone in needing its 16 columns of H, so those go from memory to registers; what all wavefronts
// need (dZ, and the scattered CBSR) goes through LDS.  Partial sums go to scratch and are added by a second kernel in a fixed order.
// What bounds it is issue: vector and matrix instructions of a SIMD's two wavefronts take turns for the most part, and a chunk has
// 144 matrix and 469 vector instructions per wavefront (counters; cells, D = 128).  1.2 M cells of D = 128: 775 -> 673 us (3.3 TB/s) with
// 576 -> 469 vector instructions (small sums are cut to finite numbers only where an operand calls for it), three chains of small
// products instead of two and one, and matrix instructions issued first; without any loads it takes 504.
// ---------------------------------------------------------------------------------------------------
template <int D> struct WTile {
    using T = Tile<D>;
    static constexpr int RGN = T::THREADS / D;         // row groups of 8 rows in a chunk
    static constexpr int CR = 8 * RGN;                 // rows per chunk: 32, or 64 / 128 for narrow D
    static constexpr int KG = RGN / 4;                 // wavefronts that share output columns: each takes 32 rows of the chunk
    static constexpr int PLANE = RGN * D;              // units per part
    static constexpr int OPER = 3 * PLANE;
    static constexpr int TPR = D == 32 ? 4 : 8;        // threads per CBSR row: a wavefront owns whole row groups
    static_assert(KG == T::RG && CR * TPR <= T::THREADS, "chunk shape");
};

struct WgradSeg {                 // one side of one graph
    const float *dY, *H1, *H2, *vals;     // H2, mask: cells only
    const uint8_t* mask;
    const uint16_t* idx;
    float* scratch;               // [products][wgs * KG][D * D]
    float* dW[3];                 // H1's, CBSR's, H2's
    int rows, k, wg0, wgs;
};
template <int G> struct WgradArgs {           // of up to G graphs
    WgradSeg s[2 * G];
    PartialSum* table;            // where the sums to be made are listed; null: wgrad_reduce_kernel follows
    int n;
};
static_assert(sizeof(WgradArgs<kMaxGraphs>) < 4096, "kernel arguments");

// The small sums are cut to finite numbers (as with_small does) in chunks that hold a number of kWide or more: below it a small sum
// is less than 32 * 5 * 2^(2 * 62 - 9) and finite.  A not-a-number needs no cut: it makes the leading sum one as well.  Cut always (96
// vector instructions, 18 to find out), 1.2 M cells and 250 000 take 0.7 and 1.6 % longer (backward passes 2 512 / 2 500, 532 / 523 us); left to a
// second walk of the workgroups whose sums are not finite, a single infinity cost 2 500 -> 2 790 and 523 -> 640.
constexpr float kWide = 4611686018427387904.0f;         // 2^62
// the largest of m >= 0, |a| and |b|, not-a-numbers aside
__device__ __forceinline__ float largest(float m, float a, float b) {
    float v;
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(v) : "v"(m), "v"(a), "v"(b));
    return v;
}
__device__ __forceinline__ float largest(const float (&x)[8], float m = 0.0f) {
#pragma unroll
    for (int j = 0; j < 8; j += 2) m = largest(m, x[j], x[j + 1]);
    return m;
}
__device__ __forceinline__ f32x4 cut_to_finite(const f32x4& x) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = __builtin_amdgcn_fmed3f(x[r], -kFloatMax, kFloatMax);
    return v;
}

template <int D, bool CELL>
__device__ __forceinline__ void wgrad_side(const DRC_CONST WgradSeg* g, bf16x8* smem, int wg) {
    using T = Tile<D>;
    using W = WTile<D>;
    constexpr int NP = CELL ? 3 : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mb = wave % T::NB, kg = wave / T::NB;
    const int col = tid % D, rgi = tid / D;                        // this thread's unit of a dense operand
    const int prow = tid / W::TPR, ppart = tid % W::TPR;
    const bool pairs = wave * 64 < W::CR * W::TPR;                 // whole wavefronts
    const int hrow = (4 * kg + (lane >> 4)) * 8, hcol = 16 * mb + (lane & 15);   // this lane's unit of the H operands

    f32x4 acc[NP][T::NB];
    int* const wide = reinterpret_cast<int*>(smem + 6 * W::OPER);      // per LDS buffer: the last chunk in it with a number of kWide or more
    if (tid < 2) wide[tid] = -1;
    __syncthreads();

    float y[8], h1[8], h2[8];
    uint32_t mk[8];
    PairRegs pr;
    const int yoff = opaque((rgi * 8 * D + col) * 4), moff = opaque(rgi * 8 * D + col), hoff = opaque((hrow * D + hcol) * 4);
    auto load_y = [&](int chunk) {                // past the last chunk: reads nothing
        const int base = chunk * W::CR, left = g->rows - base;
        const Buf by = block_view(g->dY + (size_t)base * D, left, D * 4);
        const Buf bm = block_view(g->mask + (size_t)base * D, left, D);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            y[j] = load1(by, yoff + j * D * 4);
            if constexpr (CELL) mk[j] = __builtin_amdgcn_raw_buffer_load_b8(bm, moff + j * D, 0, kNt);
        }
        load_pairs<W::TPR>(pr, block_view(g->vals + (size_t)base * g->k, left, g->k * 4), block_view(g->idx + (size_t)base * g->k, left, g->k * 2),
                           g->k, prow, ppart);
    };
    auto load_h = [&](int chunk) {
        const int base = chunk * W::CR, left = g->rows - base;
        const Buf b1 = block_view(g->H1 + (size_t)base * D, left, D * 4);
        const Buf b2 = block_view(g->H2 + (size_t)base * D, left, D * 4);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            h1[j] = load1(b1, hoff + j * D * 4);
            if constexpr (CELL) h2[j] = load1(b2, hoff + j * D * 4);
        }
    };
    auto put = [&](bf16x8* oper, const Split8& s) {
#pragma unroll
        for (int p = 0; p < 3; ++p) oper[p * W::PLANE + tid] = s.p[p];          // unit (rgi, col) sits at rgi * D + col = tid
    };
    auto commit = [&](int chunk, int to) {
        bf16x8* const buf = smem + to * 3 * W::OPER;
        float most = largest(y);
        if (pairs) {
#pragma unroll
            for (int u = 0; u < kPairs; u += 2) most = largest(most, pr.v[u], pr.v[u + 1]);
        }
        if (most >= kWide) wide[to] = chunk;
        const Split8 sp = split8(y);
        if constexpr (CELL) {
            const Split8 s1 = select8(sp, [&](int j) { return mk[j] == 1u; }), s2 = select8(sp, [&](int j) { return mk[j] == 0u; });
            put(buf, s1);
            put(buf + 2 * W::OPER, s2);
        } else {
            put(buf, sp);
        }
        if (pairs) {
            // a wavefront owns whole row groups: it clears their units, then places the pairs (LDS keeps its order)
            constexpr int RGW = 64 / W::TPR / 8;                               // row groups per wavefront
            bf16x8* const opS = buf + W::OPER;
            const bf16x8 z = {};
            bf16x8* const mine = opS + wave * RGW * D + lane;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int u = 0; u < RGW * D; u += 64)
                    if (RGW * D % 64 == 0 || u + lane < RGW * D) mine[p * W::PLANE + u] = z;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            auto put_one = [&](int c, float v) {
                put_parts(reinterpret_cast<__bf16*>(opS + (prow >> 3) * D + c) + (prow & 7), 8 * W::PLANE, v);
            };
#pragma unroll
            for (int u = 0; u < kPairs; ++u)
                if (ppart + W::TPR * u < g->k) put_one((int)pr.c[u], pr.v[u]);      // rows past the end: a zero at column 0
            const int row = chunk * W::CR + prow;
            if (g->k > W::TPR * kPairs && row < g->rows)
                for (int p = ppart + W::TPR * kPairs; p < g->k; p += W::TPR) {
                    const float v = g->vals[(size_t)row * g->k + p];
                    if (__builtin_fabsf(v) >= kWide) wide[to] = chunk;
                    put_one(g->idx[(size_t)row * g->k + p], v);
                }
        }
    };
    const int chunks = (g->rows + W::CR - 1) / W::CR;
    // Matrix instructions go first: cells 700 -> 674 us; nets 357 -> 373 (two products a chunk: they wait for the staging, as cells do
    // whose selections do not fit the registers, k = 64: 184 -> 190 us at 250 000 rows).
    const bool matrix_first = CELL && g->k <= W::TPR * kPairs;
    const auto walk = [&](auto first) {
        constexpr bool kFirst = decltype(first)::value;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < T::NB; ++j) acc[p][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        int chunk = wg, cur = 0;
        if (chunk < chunks) {
            load_y(chunk);
            if constexpr (!kFirst) load_h(chunk);
            commit(chunk, 0);
            load_y(chunk + g->wgs);
            if constexpr (kFirst) load_h(chunk);          // the order in which the loop issues them
        }
        for (; chunk < chunks; chunk += g->wgs, cur ^= 1) {
            __syncthreads();                          // this chunk is in LDS; the other buffer may be overwritten
            const int next = chunk + g->wgs;
            bf16x8* const buf = smem + cur * 3 * W::OPER;
            auto stage_next = [&]() {
                if (matrix_first) __builtin_amdgcn_s_setprio(0);
                commit(next, cur ^ 1);
                load_y(next + g->wgs);
                if (matrix_first) __builtin_amdgcn_s_setprio(1);
            };
            if constexpr (kFirst) stage_next();
            __builtin_amdgcn_sched_barrier(0);
            float most = largest(h1);
            if constexpr (CELL) most = largest(h2, most);
            const Split8 a1 = split8(h1);
            Split8 a2;
            if constexpr (CELL) a2 = split8(h2);
            // H is a wavefront's own, what is staged is everybody's
            const bool cut = __builtin_amdgcn_readfirstlane(wide[cur]) == chunk || __builtin_amdgcn_ballot_w64(most >= kWide) != 0;
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 aS[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) aS[p] = buf[W::OPER + p * W::PLANE + (hrow >> 3) * D + hcol];
            // The products of this chunk are summed from zero, leading and small ones apart, and added to the running sum
            // with one rounding: inside the matrix unit they would be cut off below it, always downwards, which over
            // many chunks adds up.  (The small sum as the leading one's start costs half of these instructions and is cut off as well:
            // errors of 2e-7 became 1.5e-6 at 1.1 M rows.)
#pragma unroll
            for (int j = 0; j < T::NB; ++j) {
                constexpr int BW[5] = {2, 0, 1, 1, 0}, AW[5] = {0, 2, 1, 0, 1};
                const int ub = (hrow >> 3) * D + 16 * j + (lane & 15);
                f32x4 lo[3] = {};
                bf16x8 b[3], b2[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    b[p] = buf[p * W::PLANE + ub];
                    if constexpr (CELL) b2[p] = buf[2 * W::OPER + p * W::PLANE + ub];
                }
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    lo[0] = mfma(b[BW[i]], a1.p[AW[i]], lo[0]);
                    lo[1] = mfma(b[BW[i]], aS[AW[i]], lo[1]);
                    if constexpr (CELL) lo[2] = mfma(b2[BW[i]], a2.p[AW[i]], lo[2]);
                }
                const f32x4 zero = {};
                f32x4 hi[3];
                hi[0] = mfma(b[0], a1.p[0], zero);
                hi[1] = mfma(b[0], aS[0], zero);
                if constexpr (CELL) hi[2] = mfma(b2[0], a2.p[0], zero);
                if (cut) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) lo[p] = cut_to_finite(lo[p]);
                }
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    acc[p][j] += hi[p] + lo[p];
                    asm volatile("" : "+v"(acc[p][j]));       // added here: the compiler would keep all sums to the end of the loop
                }
                __builtin_amdgcn_sched_barrier(0);    // one column block's operands at a time: more do not fit the registers
            }
            load_h(next);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!kFirst) stage_next();
        }
    };
    if (wave < T::WAVES / 2) walk(yes{});
    else walk(no{});
    __builtin_amdgcn_s_setprio(0);
    // lane: row 16 mb + (lane & 15) of dW, columns 16 j + 4 (lane >> 4) ..
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        float* out = g->scratch + ((size_t)p * g->wgs * W::KG + (size_t)wg * W::KG + kg) * D * D;
#pragma unroll
        for (int j = 0; j < T::NB; ++j)
            *reinterpret_cast<f32x4*>(out + (size_t)(16 * mb + (lane & 15)) * D + 16 * j + 4 * (lane >> 4)) = acc[p][j];
    }
}

template <int D, typename ARGS> __device__ __forceinline__ void wgrad_workgroup(const DRC_CONST ARGS* k, bf16x8* smem, int wg) {
    if (k->table && wg == 0 && (int)threadIdx.x < k->n / 2 * kSumsPerGraph) {      // cells and nets in turn
        const int q = threadIdx.x / kSumsPerGraph, e = threadIdx.x % kSumsPerGraph, prod = e < 3 ? e : e - 3;
        const DRC_CONST WgradSeg* const g = k->s + 2 * q + (e < 3 ? 0 : 1);
        const int n = g->wgs * WTile<D>::KG;
        k->table[threadIdx.x] = PartialSum{g->scratch + (size_t)prod * n * D * D, g->dW[prod], n, D * D};
    }
    int q = 0;
    while (q + 1 < k->n && wg >= k->s[q + 1].wg0) ++q;
    const DRC_CONST WgradSeg* const g = k->s + q;
    if (g->mask) wgrad_side<D, true>(g, smem, wg - g->wg0);
    else wgrad_side<D, false>(g, smem, wg - g->wg0);
}
template <int D>
__global__ __launch_bounds__(Tile<D>::THREADS, 2) void wgrad_partial_kernel(WgradArgs<kMaxGraphs> a) {
    extern __shared__ bf16x8 smem8[];
    wgrad_workgroup<D>(kernel_args<WgradArgs<kMaxGraphs>>(), smem8, blockIdx.x);
}

// Weight gradients and projections of a backward pass in one launch.  Neither waits for the other, and while either has fewer tiles
// than the chip has compute units, or ends in a last round that is half empty, the other's workgroups fill it.  Two launches / one,
// whole layers, us: 2 048 cells, D = 64 60 / 50; 10 000 82 / 76; 60 000 185 / 179; 20 000, D = 128 194 / 187; 250 000 1 182 / 1 172.
constexpr int kBothGraphs = 12;
struct DenseBwdArgs {
    ProjBwdArgs<kBothGraphs> proj;
    WgradArgs<kBothGraphs> wgrad;
    int wgrad_wgs;
};
static_assert(sizeof(DenseBwdArgs) < 4096, "kernel arguments");
template <int D>
__global__ __launch_bounds__(Tile<D>::THREADS, 2) void dense_bwd_kernel(DenseBwdArgs a) {
    extern __shared__ bf16x8 smem8[];
    const DRC_CONST DenseBwdArgs* const k = kernel_args<DenseBwdArgs>();
    const int wg = (int)blockIdx.x - k->wgrad_wgs;
    if (wg < 0) wgrad_workgroup<D>(&k->wgrad, smem8, blockIdx.x);
    else if (wg < k->proj.cell_wgs) proj_bwd_side<D, true>(&k->proj, smem8, wg, k->proj.cell_wgs);
    else proj_bwd_side<D, false>(&k->proj, smem8, wg - k->proj.cell_wgs, k->proj.net_wgs);
}

// dW[i] = sum over a side's partials in a fixed order: wavefront w of the workgroup sums partials w, w + 16, ... of 64 x 4
// consecutive entries, then the 16 sums are added in order.  In 64 bits: up to 1024 partials of nearly equal size lose as much
// in 32-bit sums as everything before.  One launch for all products of all sides and graphs.
constexpr int kRedWaves = 16;
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <int D>
__global__ __launch_bounds__(64 * kRedWaves) void wgrad_reduce_kernel(WgradArgs<kMaxGraphs> a) {
    __shared__ f64x4 part[kRedWaves][64];
    constexpr int kBlocks = D * D / 256;                 // workgroups per product
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int job = blockIdx.x / kBlocks, q = job / 3, prod = job % 3;
    const WgradSeg& g = a.s[q];
    if (g.dW[prod] == nullptr) return;
    const int n = g.wgs * WTile<D>::KG;
    const int at = (blockIdx.x % kBlocks) * 256 + 4 * lane;
    const float* src = g.scratch + (size_t)prod * n * D * D + at;
    f64x4 s = {0., 0., 0., 0.};
    int b = wave;
    for (; b + 3 * kRedWaves < n; b += 4 * kRedWaves) {  // four loads in flight
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4*>(src + (size_t)(b + u * kRedWaves) * D * D);
#pragma unroll
        for (int u = 0; u < 4; ++u) s += __builtin_convertvector(v[u], f64x4);
    }
    for (; b < n; b += kRedWaves) s += __builtin_convertvector(*reinterpret_cast<const f32x4*>(src + (size_t)b * D * D), f64x4);
    part[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
        f64x4 t = part[0][lane];
#pragma unroll
        for (int w = 1; w < kRedWaves; ++w) t += part[w][lane];
        float* o = g.dW[prod] + at;                      // weight gradients need not be 16-byte aligned
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (float)((double)kUnscale * t[r]);
    }
}

// ---------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------
// raises a kernel's LDS limit, once per device, and returns how many of its workgroups fit the chip
template <typename K> static int resident(K kernel, int threads, size_t lds, PerDevice& cache, int* out) {
    int dev = 0;
    DRC_HIP(hipGetDevice(&dev));
    return cache.get(dev, out, [&](int* n) -> int {
        DRC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        int per_cu = 0, cus = 0;
        DRC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds));
        DRC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        *n = (per_cu < 1 ? 1 : per_cu) * cus;
        return DR_OK;
    });
}

// Workgroups of the two sides: in proportion to their work (three and two products per row), all of them resident.
static void share(int64_t cell_work, int64_t net_work, int cell_tiles, int net_tiles, int res, int* cells, int* nets) {
    if (cell_tiles + net_tiles <= res) { *cells = cell_tiles; *nets = net_tiles; return; }
    int64_t c = (cell_work * res + (cell_work + net_work) / 2) / (cell_work + net_work);
    if (c < 1 && cell_tiles) c = 1;
    if (c > res - 1 && net_tiles) c = res - 1;
    if (!cell_tiles) c = 0;
    if (c > cell_tiles) c = cell_tiles;
    *cells = (int)c;
    int64_t n = res - c;
    if (n > net_tiles) n = net_tiles;
    *nets = (int)n;
}

template <int D, int CP> static int launch_proj_fwd_cp(ProjFwdArgs& a, hipStream_t s) {
    using T = Tile<D>;
    static PerDevice cache;
    constexpr size_t lds = sizeof(bf16x8) * 2 * 3 * T::OPER;
    int res = 0;
    DRC_TRY(resident(&proj_kernel<D, CP>, T::THREADS, lds, cache, &res));
    a.cell_tiles = a.net_tiles = 0;
    for (int i = 0; i < a.n; ++i) {
        a.cell[i].tile0 = a.cell_tiles; a.net[i].tile0 = a.net_tiles;
        a.cell_tiles += (a.cell[i].rows + T::BM - 1) / T::BM;
        a.net_tiles += (a.net[i].rows + T::BM - 1) / T::BM;
    }
    int nets = 0;
    share(3ll * a.cell_tiles, 2ll * a.net_tiles, a.cell_tiles, a.net_tiles, res, &a.cell_wgs, &nets);
    if (a.cell_wgs + nets == 0) return DR_OK;
    hipLaunchKernelGGL((proj_kernel<D, CP>), dim3((unsigned)(a.cell_wgs + nets)), dim3(T::THREADS), lds, s, a);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

template <int D> static int launch_proj_fwd_d(ProjFwdArgs& a, hipStream_t s) {
    int64_t rows = 0;
    for (int i = 0; i < a.n; ++i) rows += (int64_t)a.cell[i].rows + a.net[i].rows;
    return rows * D * 4 > kL2Bytes ? launch_proj_fwd_cp<D, 0>(a, s) : launch_proj_fwd_cp<D, kNt>(a, s);
}

int launch_proj_fwd(const ProjFwdJob* jobs, int n, const dr_heteroconv_weights& W, int D, bool relu, hipStream_t s) {
    if (n > kMaxGraphs) return fail(DR_ERR_INVALID_ARG, "projection of %d graphs in one launch", n);
    ProjFwdArgs a{};
    a.n = n;
    a.relu = relu ? 1 : 0;
    a.w_self_near = W.self_near; a.w_neigh_near = W.neigh_near; a.w_pinned = W.pinned;
    a.w_self_pins = W.self_pins; a.w_neigh_pins = W.neigh_pins;
    for (int i = 0; i < n; ++i) {
        const ProjFwdJob& j = jobs[i];
        a.cell[i] = ProjFwdSide{j.vals_near, j.H_near, j.H_pinned, j.idx_near, j.Y_cell, j.mask, (int)j.Nc, j.k_near, 0};
        a.net[i] = ProjFwdSide{j.vals_self, j.H_pins, nullptr, j.idx_self, j.Y_net, nullptr, (int)j.Nn, j.k_self, 0};
    }
    switch (D) {
        case 32: return launch_proj_fwd_d<32>(a, s);
        case 64: return launch_proj_fwd_d<64>(a, s);
        case 96: return launch_proj_fwd_d<96>(a, s);
        case 128: return launch_proj_fwd_d<128>(a, s);
        default: return fail(DR_ERR_UNSUPPORTED, "projection width D = %d not in {32,64,96,128}", D);
    }
}

template <int D> constexpr size_t dproj_lds() {
    return sizeof(bf16x8) * 4 * Tile<D>::OPER + sizeof(float) * 2 * Tile<D>::BM * (D + 4);
}
// tiles and workgroups, `res` at most
template <int D, int G> static void plan_proj_bwd(ProjBwdArgs<G>& a, int res) {
    using T = Tile<D>;
    a.cell_tiles = a.net_tiles = 0;
    for (int i = 0; i < a.n; ++i) {
        a.cell[i].tile0 = a.cell_tiles; a.net[i].tile0 = a.net_tiles;
        a.cell_tiles += (a.cell[i].rows + T::BM - 1) / T::BM;
        a.net_tiles += (a.net[i].rows + T::BM - 1) / T::BM;
    }
    share(3ll * a.cell_tiles, 2ll * a.net_tiles, a.cell_tiles, a.net_tiles, res, &a.cell_wgs, &a.net_wgs);
}
template <int G> static void set_proj_bwd(ProjBwdArgs<G>& a, const ProjBwdJob* jobs, int n, const dr_heteroconv_weights& W) {
    a.n = n;
    a.w_self_near = W.self_near; a.w_neigh_near = W.neigh_near; a.w_pinned = W.pinned;
    a.w_self_pins = W.self_pins; a.w_neigh_pins = W.neigh_pins;
    for (int i = 0; i < n; ++i) {
        const ProjBwdJob& j = jobs[i];
        a.cell[i] = ProjBwdSide{j.dY_cell, j.mask, j.dH_near, j.dH_pinned, j.idx_near, j.S_cell, (int)j.Nc, j.k_near, 0};
        a.net[i] = ProjBwdSide{j.dY_net, nullptr, j.dH_pins, nullptr, j.idx_self, j.S_net, (int)j.Nn, j.k_self, 0};
    }
}
template <int D> static int launch_proj_bwd_d(ProjBwdArgs<kMaxGraphs>& a, hipStream_t s) {
    using T = Tile<D>;
    static PerDevice cache;
    int res = 0;
    DRC_TRY(resident(&dproj_kernel<D>, T::THREADS, dproj_lds<D>(), cache, &res));
    plan_proj_bwd<D>(a, res);
    if (a.cell_wgs + a.net_wgs == 0) return DR_OK;
    hipLaunchKernelGGL((dproj_kernel<D>), dim3((unsigned)(a.cell_wgs + a.net_wgs)), dim3(T::THREADS), dproj_lds<D>(), s, a);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_proj_bwd(const ProjBwdJob* jobs, int n, const dr_heteroconv_weights& W, int D, hipStream_t s) {
    if (n > kMaxGraphs) return fail(DR_ERR_INVALID_ARG, "projection of %d graphs in one launch", n);
    ProjBwdArgs<kMaxGraphs> a{};
    set_proj_bwd(a, jobs, n, W);
    switch (D) {
        case 32: return launch_proj_bwd_d<32>(a, s);
        case 64: return launch_proj_bwd_d<64>(a, s);
        case 96: return launch_proj_bwd_d<96>(a, s);
        case 128: return launch_proj_bwd_d<128>(a, s);
        default: return fail(DR_ERR_UNSUPPORTED, "projection width D = %d not in {32,64,96,128}", D);
    }
}

template <int D> static int64_t wgrad_chunks(int64_t rows) { return (rows + WTile<D>::CR - 1) / WTile<D>::CR; }
template <int D> static size_t wgrad_bytes_d(int64_t rows, int products) {
    return sizeof(float) * products * (size_t)wgrad_most(wgrad_chunks<D>(rows)) * WTile<D>::KG * D * D;
}
size_t wgrad_scratch_bytes(int64_t rows, int D, int products) {
    switch (D) {
        case 32: return wgrad_bytes_d<32>(rows, products);
        case 64: return wgrad_bytes_d<64>(rows, products);
        case 96: return wgrad_bytes_d<96>(rows, products);
        default: return wgrad_bytes_d<128>(rows, products);
    }
}

template <int D> constexpr size_t wgrad_lds() { return sizeof(bf16x8) * (2 * 3 * WTile<D>::OPER + 1); }
// workgroups of every side; returns their number
template <int D, int G> static int plan_wgrad(WgradArgs<G>& a, int res) {
    WgradSide sides[2 * G];
    for (int i = 0; i < a.n; ++i) sides[i] = WgradSide{a.s[i].rows, a.s[i].mask ? 3 : 2};
    int wgs = 0;
    for (int i = 0; i < a.n; ++i) {
        WgradSeg& g = a.s[i];
        g.wgs = wgrad_share(sides, a.n, i, D, WTile<D>::CR, res, kFullLaunch);
        g.wg0 = wgs;
        wgs += g.wgs;
    }
    return wgs;
}
template <int G> static void set_wgrad(WgradArgs<G>& a, const WgradJob* jobs, int n) {
    a.n = n;
    for (int i = 0; i < n; ++i) {
        const WgradJob& j = jobs[i];
        a.s[i] = WgradSeg{j.dY, j.H1, j.H2, j.vals, j.mask, j.idx, static_cast<float*>(j.scratch), {j.dW_H1, j.dW_cbsr, j.dW_H2},
                          (int)j.rows, j.k, 0, 0};
    }
}
template <int D> static int launch_wgrad_d(WgradArgs<kMaxGraphs>& a, hipStream_t s) {
    using T = Tile<D>;
    static PerDevice cache;
    int res = 0;
    DRC_TRY(resident(&wgrad_partial_kernel<D>, T::THREADS, wgrad_lds<D>(), cache, &res));
    const int wgs = plan_wgrad<D>(a, res);
    hipLaunchKernelGGL((wgrad_partial_kernel<D>), dim3((unsigned)wgs), dim3(T::THREADS), wgrad_lds<D>(), s, a);
    if (!a.table) hipLaunchKernelGGL((wgrad_reduce_kernel<D>), dim3((unsigned)(a.n * 3 * (D * D / 256))), dim3(64 * kRedWaves), 0, s, a);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

static int launch_wgrads_to(const WgradJob* jobs, int n, int D, PartialSum* table, hipStream_t s) {
    if (n > 2 * kMaxGraphs) return fail(DR_ERR_INVALID_ARG, "weight gradients of %d operands in one launch", n);
    WgradArgs<kMaxGraphs> a{};
    set_wgrad(a, jobs, n);
    a.table = table;
    if (n == 0) return DR_OK;
    switch (D) {
        case 32: return launch_wgrad_d<32>(a, s);
        case 64: return launch_wgrad_d<64>(a, s);
        case 96: return launch_wgrad_d<96>(a, s);
        case 128: return launch_wgrad_d<128>(a, s);
        default: return fail(DR_ERR_UNSUPPORTED, "projection width D = %d not in {32,64,96,128}", D);
    }
}
int launch_wgrads(const WgradJob* jobs, int n, int D, hipStream_t s) { return launch_wgrads_to(jobs, n, D, nullptr, s); }

template <int D> static int launch_dense_bwd_d(const WgradJob* wgrads, const ProjBwdJob* proj, int n, const dr_heteroconv_weights& W,
                                               PartialSum* table, hipStream_t s) {
    if (n > kBothGraphs) {
        DRC_TRY(launch_wgrads_to(wgrads, 2 * n, D, table, s));
        return launch_proj_bwd(proj, n, W, D, s);
    }
    using T = Tile<D>;
    static PerDevice cache;
    constexpr size_t lds = dproj_lds<D>() > wgrad_lds<D>() ? dproj_lds<D>() : wgrad_lds<D>();
    int res = 0;
    DRC_TRY(resident(&dense_bwd_kernel<D>, T::THREADS, lds, cache, &res));
    DenseBwdArgs a{};
    set_proj_bwd(a.proj, proj, n, W);
    set_wgrad(a.wgrad, wgrads, 2 * n);
    a.wgrad.table = table;
    // As many workgroups for either as it would have alone: how the weight gradients of a pass are summed does not depend on the
    // projections beside them.  (It does on the other sides of the pass: they share the workgroups, wgrad_share.)
    plan_proj_bwd<D>(a.proj, res);
    a.wgrad_wgs = plan_wgrad<D>(a.wgrad, res);
    hipLaunchKernelGGL((dense_bwd_kernel<D>), dim3((unsigned)(a.wgrad_wgs + a.proj.cell_wgs + a.proj.net_wgs)), dim3(T::THREADS), lds, s, a);
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_dense_bwd(const WgradJob* wgrads, const ProjBwdJob* proj, int n, const dr_heteroconv_weights& W, int D, PartialSum* table,
                     PendingSums* pending, hipStream_t s) {
    if (n > kMaxGraphs) return fail(DR_ERR_INVALID_ARG, "dense gradients of %d graphs in one launch", n);
    *pending = PendingSums{table, n * kSumsPerGraph, D * D};
    switch (D) {
        case 32: return launch_dense_bwd_d<32>(wgrads, proj, n, W, table, s);
        case 64: return launch_dense_bwd_d<64>(wgrads, proj, n, W, table, s);
        case 96: return launch_dense_bwd_d<96>(wgrads, proj, n, W, table, s);
        case 128: return launch_dense_bwd_d<128>(wgrads, proj, n, W, table, s);
        default: return fail(DR_ERR_UNSUPPORTED, "projection width D = %d not in {32,64,96,128}", D);
    }
}

}  // namespace drc
