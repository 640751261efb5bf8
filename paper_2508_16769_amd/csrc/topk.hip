// D-ReLU (paper Section 3.1): per row keep the k largest signed values, ties to the lowest column,
// survivors written in ascending column order as CBSR (vals, idx).
//
// Two kernels: topk_groups_kernel, several rows per wavefront, for rows of up to 128 columns in whole float4s; and
// topk_rows_kernel for everything else and for the rank order:
// one wavefront owns one row at a time.  Lane l holds columns l, 64+l, 128+l, ... (coalesced dword
// loads).  Values are mapped to order-preserving unsigned keys; the k-th largest key is found by a
// most-significant-bit-first search in which every step is one v_cmp per register plus a scalar
// popcount of the ballot, started below the previous row's sign and exponent bits when two probes confirm
// them, and with an early exit once a probe isolates exactly k elements; compaction
// positions come from mbcnt prefix counts of the keep-ballots, which yields ascending column order for
// free.  A row that is needed at two widths (one K per edge type) is loaded once and selected twice.
// The rank-ordered variant (largest value first; every smaller selection is a prefix, which degree-adaptive
// K relies on) stages the kept keys of a row in LDS in column order and lets every kept element count the
// keys that precede it: greater, or equal with a lower column.
#include "dr_internal.h"

#include <cmath>
#include <type_traits>

namespace drc {

__device__ __forceinline__ uint32_t order_key(float v) {
    uint32_t u = __float_as_uint(v);
    u = (u == 0x80000000u) ? 0u : u;                    // -0.0 ties with +0.0
    // larger float <=> larger key; all keys of numbers > 0 (that of the not-a-number 0xffffffff is 0).  Negative values flip every bit, the others the sign bit only
    // (written without a branch: the scalar unit is what bounds this kernel).
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr int kRowsInFlight = 4;   // rows whose loads are outstanding per wavefront

// Where the k-th largest of D standard normal numbers lies, and how far apart they are there.
struct FirstGuess { float z, gap; };
static FirstGuess first_guess(int D, int k) {
    const double p = 1.0 - (k - 0.5) / D, z = 4.91 * (std::pow(p, 0.14) - std::pow(1.0 - p, 0.14));     // Tukey's lambda: to 0.01
    return FirstGuess{(float)z, (float)(2.5066 * std::exp(0.5 * z * z) / D)};
}

struct TopkSeg {                   // one embedding matrix of a launch
    const float* X;
    float *vals, *vals2;           // vals2 / idx2: a second selection of the same rows, or null
    uint16_t *idx, *idx2;
    int n, k, k2, blk0, n_blocks;  // workgroups [blk0, blk0 + n_blocks)
    int wide_out;                  // the outputs take 16-byte (values) and 8-byte (columns) stores
    FirstGuess guess, guess2;
};
constexpr int kTopkSegs = 32;
struct TopkArgs { TopkSeg s[kTopkSegs]; int n, D, k_max; };
static_assert(sizeof(TopkArgs) < 4096, "kernel arguments");

template <int EPL, bool DUAL, bool RANKED>
__global__ __launch_bounds__(256) void topk_rows_kernel(TopkArgs args) {
    extern __shared__ uint4 kept_keys4[];                     // RANKED: [4 wavefronts][k rounded up to 4] keys of the current row
    int sg = 0;
    while (sg + 1 < args.n && (int)blockIdx.x >= args.s[sg + 1].blk0) ++sg;
    const TopkSeg& seg = args.s[sg];
    const float* __restrict__ X = seg.X;
    float* __restrict__ vals = seg.vals;
    uint16_t* __restrict__ idx = seg.idx;
    const int n = seg.n, D = args.D, k = seg.k;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int k4 = (k + 3) >> 2;
    uint32_t* const my_keys = reinterpret_cast<uint32_t*>(kept_keys4 + wave * k4);
    const int stride = seg.n_blocks * (blockDim.x >> 6);     // rows between consecutive rows of one wavefront
    const int row0 = (blockIdx.x - seg.blk0) * (blockDim.x >> 6) + wave;

    // loads are unconditional (row and column clamped to valid addresses): the next rows stay in flight
    // while the current one is selected
    float v[kRowsInFlight][EPL];
    auto load_row = [&](float (&dst)[EPL], int row) {
        const float* x = X + (size_t)min(row, n - 1) * D;
#pragma unroll
        for (int s = 0; s < EPL; ++s) dst[s] = __builtin_nontemporal_load(x + min(s * kWave + lane, D - 1));   // read once
    };
    uint32_t hint = 0, hint2 = 0;                             // thresholds of the previous row of this wavefront
    auto select_row = [&](const float (&val)[EPL], int row, int k, float* __restrict__ vals, uint16_t* __restrict__ idx,
                          uint32_t& t_hint) {
        uint32_t key[EPL];
#pragma unroll
        for (int s = 0; s < EPL; ++s) {
            const uint32_t real = order_key(val[s]);
            key[s] = (s * kWave + lane < D) ? real : 0u;      // padding key 0 < real keys
        }
        // T = largest threshold with count(key >= T) >= k  == the k-th largest key.  The search stops as
        // soon as a probe separates exactly k elements: then {key >= T} is already the answer, which on
        // tie-free data happens after about a dozen of the 32 bits.
        // The sign and exponent bits of T rarely change from one row to the next: probe the previous row's
        // leading nine bits first (two counts) and, if T does lie in that binade, search only below them.
        uint32_t T = 0;
        int top = 31;
        {
            // (for finite inputs a threshold never lies in the last binade; if hi did wrap to 0, c_hi would count
            // every element and the full search below would run)
            const uint32_t lo = t_hint & 0xff800000u, hi = lo + 0x00800000u;
            int c_lo = 0, c_hi = 0;
#pragma unroll
            for (int s = 0; s < EPL; ++s) {
                c_lo += __popcll(__builtin_amdgcn_ballot_w64(key[s] >= lo));
                c_hi += __popcll(__builtin_amdgcn_ballot_w64(key[s] >= hi));
            }
            if (c_lo >= k && c_hi < k) {
                T = lo;
                top = (c_lo == k) ? -1 : 22;          // exactly k at or above the binade's floor: done
            }
        }
        for (int bit = top; bit >= 0; --bit) {
            uint32_t cand = T | (1u << bit);
            int cnt = 0;
#pragma unroll
            for (int s = 0; s < EPL; ++s) cnt += __popcll(__builtin_amdgcn_ballot_w64(key[s] >= cand));
            if (cnt >= k) T = cand;
            if (cnt == k) break;
        }
        t_hint = T;
        int n_gt = 0;
#pragma unroll
        for (int s = 0; s < EPL; ++s) n_gt += __popcll(__builtin_amdgcn_ballot_w64(key[s] > T));
        const int need_eq = k - n_gt;                   // >= 1 ties to take, lowest columns first
        int kept_before = 0, eq_before = 0;
        const size_t base = (size_t)row * k;
        bool keep_s[EPL];
        int pos_s[EPL];
#pragma unroll
        for (int s = 0; s < EPL; ++s) {
            bool gt = key[s] > T;
            bool eq = key[s] == T;
            unsigned long long meq = __builtin_amdgcn_ballot_w64(eq);
            const bool tie_taken = (eq_before + lanes_below(meq)) < need_eq;     // evaluated by every lane: no branch
            const bool keep = gt || (eq && tie_taken);
            unsigned long long mk = __builtin_amdgcn_ballot_w64(keep);
            const int pos = kept_before + lanes_below(mk);     // position in ascending column order
            kept_before += __popcll(mk);
            eq_before += __popcll(meq);
            if constexpr (!RANKED) {
                if (keep) {                                    // stored at once: the predicate stays a lane mask
                    vals[base + pos] = val[s];
                    idx[base + pos] = (uint16_t)(s * kWave + lane);
                }
            } else {
                keep_s[s] = keep;
                pos_s[s] = pos;
            }
        }
        if constexpr (RANKED) {
            // One wavefront executes its LDS accesses in program order, so the reads below see the keys written here
            // and the next row's writes come after this row's reads; the fences keep the compiler from reordering.
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            if (lane < 4 * k4 - k) my_keys[k + lane] = 0u;     // padding keys: below every real key, so they never count
#pragma unroll
            for (int s = 0; s < EPL; ++s)
                if (keep_s[s]) my_keys[pos_s[s]] = key[s];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = 0; s < EPL; ++s) {
                if (!keep_s[s]) continue;
                const uint32_t mine = key[s];
                const int p_me = pos_s[s];
                int rank = 0;
                for (int p4 = 0; p4 < k4; ++p4) {              // every lane reads the same 16 bytes: broadcast
                    const uint4 o = reinterpret_cast<const uint4*>(my_keys)[p4];
                    const int p = 4 * p4;
                    rank += (o.x > mine || (o.x == mine && p + 0 < p_me)) ? 1 : 0;
                    rank += (o.y > mine || (o.y == mine && p + 1 < p_me)) ? 1 : 0;
                    rank += (o.z > mine || (o.z == mine && p + 2 < p_me)) ? 1 : 0;
                    rank += (o.w > mine || (o.w == mine && p + 3 < p_me)) ? 1 : 0;
                }
                vals[base + rank] = val[s];
                idx[base + rank] = (uint16_t)(s * kWave + lane);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };

#pragma unroll
    for (int i = 0; i < kRowsInFlight; ++i) load_row(v[i], row0 + i * stride);
    for (int base = row0; base < n; base += kRowsInFlight * stride) {
#pragma unroll
        for (int i = 0; i < kRowsInFlight; ++i) {
            const int row = base + i * stride;
            if (row < n) {
                select_row(v[i], row, k, vals, idx, hint);
                if constexpr (DUAL) {
                    if (seg.vals2) select_row(v[i], row, seg.k2, seg.vals2, seg.idx2, hint2);
                }
            }
            load_row(v[i], row + kRowsInFlight * stride);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Rows of up to 128 columns, whole float4s: several rows per wavefront.
//
// L lanes share a row; lane t holds the columns 4u .. 4u+3 of its units u = t, t + L, ... (SLOTS float4 loads, each of which
// reads whole lines).  With one row per wavefront (topk_rows_kernel) a probe of the search costs an instruction of the vector
// and several of the scalar unit per row, and both were busy three quarters of the time; here a probe counts 64 / L rows at
// once: two vector instructions per element and a few lane exchanges, nothing scalar.
//   Search for T, the k-th largest key.  The first probe is where T would lie if the row's values were normally distributed
// (from their mean and variance), the next ones follow the density of values that goes with it or the bracket's linear
// interpolation, until every row of the wavefront is within kWalk of k keys; from there a row goes up or down key by key (the
// nearest key above and below take a subtraction and half a three-way minimum and maximum per element, a probe two instructions).
// Probing to the end would take as many probes as the slowest of the rows: 8.1 on average for eight rows of 128 normal values
// with k = 32, where under 2 probes and 4 steps do.  (A guess from the rows before instead: 2 to 6 % slower, and no guess at all
// where the scale changes.)  Rows that are still far after kGuided probes (skewed data) go on with a bracket in key space,
// halved and interpolated in turn, whose ends are moved to keys of the row, so that few distinct values take few probes; and
// when the number of keys that would be kept is not k (equal keys were walked over), that search goes on to the end.  A wavefront
// whose rows needed that from far away begins its later trips where T was, drifting with it, for as long as this serves.
//   Ties at T are told apart in a branch of their own (by clearing the keys that lose), so the usual row does not pay.
//   Compaction.  The kept counts of a lane's slots travel as four bytes of one register through one scan over the lanes.  Kept
// (value, column) pairs are placed in LDS, and the rows' pairs, which lie behind one another in memory, leave as whole
// 16- and 8-byte stores.
// At D = 128 the vector units are 93-96 % busy while the rows move at 5.0 TB/s, what a plain copy reaches: 1.2 M and 0.9 M rows,
// k = 32, together 368 -> 291 us; 430 000 rows 91 -> 64 us.  At D = 64
// still by its instructions: 100 000 rows, k = 16, 22 -> 13 us; 3072 rows 5.4 -> 3.9 us; two selections at D = 96, 58 000 rows,
// 32 -> 18 us.  Other data, one row per wavefront / now (k = 32, D = 128): 1.2 M rows normal 226 -> 197 us,
// exp(2 N) 270 -> 242 (305 without the trace), uniform with 2 % outliers of 1e6 210 -> 184 (335), Cauchy 254 -> 216 (300), two narrow
// peaks 253 -> 184 (303); 250 000 rows, values rounded to halves 128 -> 87, zeros and ones 116 -> 64, outliers 53 -> 54, exp(2 N)
// 65 -> 60.  Where wavefronts have one trip only (65 000 rows at this width) such rows cost more than with a wavefront each:
// 20 000 rows with outliers 8.5 -> 11.3, Cauchy 9.5 -> 10.0; 45 677 x 100 with outliers 14.3 -> 18.0.
// ---------------------------------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ uint32_t lane_swap(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
// sum over the L lanes of a group, in every lane
template <int L> __device__ __forceinline__ uint32_t group_sum(uint32_t v) {
    v += lane_swap<kQuadXor1>(v);
    v += lane_swap<kQuadXor2>(v);
    if constexpr (L >= 8) v += lane_swap<kHalfMirror>(v);
    if constexpr (L >= 16) v += lane_swap<kMirror>(v);
    return v;
}
template <int L> __device__ __forceinline__ uint32_t group_max(uint32_t v) {
    v = max(v, lane_swap<kQuadXor1>(v));
    v = max(v, lane_swap<kQuadXor2>(v));
    if constexpr (L >= 8) v = max(v, lane_swap<kHalfMirror>(v));
    if constexpr (L >= 16) v = max(v, lane_swap<kMirror>(v));
    return v;
}
// sum over the lanes of the group before this one (t: lane in the group)
template <int L> __device__ __forceinline__ uint32_t group_before(uint32_t v, int t) {
    uint32_t x = v;
    uint32_t y = lane_swap<0x111>(x);          // row_shr:1, 2, 4, 8
    x += t >= 1 ? y : 0u;
    y = lane_swap<0x112>(x);
    x += t >= 2 ? y : 0u;
    if constexpr (L >= 8) {
        y = lane_swap<0x114>(x);
        x += t >= 4 ? y : 0u;
    }
    if constexpr (L >= 16) {
        y = lane_swap<0x118>(x);
        x += t >= 8 ? y : 0u;
    }
    return x - v;
}
__device__ __forceinline__ uint32_t key_of(float v) {       // order_key in three instructions (-0 + 0 = +0)
    const uint32_t u = __float_as_uint(v + 0.0f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float value_of(uint32_t key) { return __uint_as_float(key ^ (~(uint32_t)((int32_t)key >> 31) | 0x80000000u)); }
constexpr int kGuided = 3, kWalk = 4;        // guided probes at most; distance from which keys are walked
constexpr int kGroupBlocks = 2048;           // eight workgroups per compute unit
constexpr int64_t kFewRows = 32768;
struct Guide { float at, gap; };            // where T is looked for first, and the distance between neighbouring values there
// The same from the rows of the trips before.  `lost`: a row had to go on with a bracket from far away.
struct Trace { Guide g; bool on, lost; };
typedef float float4v __attribute__((ext_vector_type(4)));

template <int L, int SLOTS> struct GroupRow {
    static constexpr int E = 4 * SLOTS;
    float v[E];
    uint32_t key[E];

    __device__ __forceinline__ void make_keys(int t, int D) {
#pragma unroll
        for (int i = 0; i < E; ++i) key[i] = 4 * (t + L * (i / 4)) < D ? key_of(v[i]) : 0u;      // what is no column counts below all
    }
    __device__ __forceinline__ uint32_t count(uint32_t cand) const {
        uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < E; ++i) c[i & 3] += key[i] >= cand ? 1u : 0u;
        return group_sum<L>((c[0] + c[1]) + (c[2] + c[3]));
    }
    // nearest key below `cand` and nearest at or above it, as distances (modulo 2^32: what lies on the other side is far away)
    __device__ __forceinline__ void neighbours(uint32_t cand, uint32_t* below, uint32_t* above) const {
        uint32_t b = 0u, a = 0xffffffffu;
#pragma unroll
        for (int i = 0; i < E; i += 2) {
            const uint32_t x = key[i] - cand, y = key[i + 1] - cand;
            b = max(b, max(x, y));
            a = min(a, min(x, y));
        }
        *below = group_max<L>(b);
        *above = ~group_max<L>(~a);
    }
    // k-th largest key, and where each slot's kept keys go (starts)
    // TRACE: 0 none, 1 notes whether one is called for, 2 follows it.
    template <int TRACE>
    __device__ __forceinline__ uint32_t threshold(int k, int t, int D, const FirstGuess& f, Trace& trace, uint32_t* at, bool* ties) {
        Guide g = TRACE == 2 && trace.on ? trace.g : guide(t, D, f);
        float lof = -__builtin_inff(), hif = __builtin_inff(), candf = g.at;
        float clo = 0.0f, chi = 0.0f;                         // counts less k
        uint32_t cand = key_of(candf);
        int d;                                                // keys at or above cand, less k
        const auto note = [&]() {
            const bool ge = d >= 0;
            lof = ge ? candf : lof;
            clo = ge ? (float)d : clo;
            hif = ge ? hif : candf;
            chi = ge ? chi : (float)d;
        };
        for (int it = 0;; ++it) {
            d = (int)count(cand) - k;
            const bool far = abs(d) > kWalk;
            if (it == kGuided - 1 || !__any(far)) break;
            note();
            const float df = (float)d;
            const float width = hif - lof;                    // infinite until both sides have been probed
            const float inside = lof + width * ((clo + 0.5f) * __builtin_amdgcn_rcpf(clo - chi + 1.0f));
            const float outside = candf + g.gap * (df + (d >= 0 ? 0.5f : -0.5f)) * (float)(it + 1);
            const float next = fabsf(width) < __builtin_inff() ? inside : outside;
            candf = far ? next : candf;
            cand = key_of(candf);
        }
        uint32_t lo = 0u, hi = 0u, kept;                      // set where they are needed: at least k keys from lo on, fewer from hi on
        bool open = abs(d) > kWalk;
        for (int reach = kWalk, trip = 0;; reach = 0) {
            if (__any(open)) {
                const bool lost = TRACE != 0 && reach != 0 && __any(abs(d) > 2 * kWalk);
                if (hi == 0u) {                               // the probes so far, else the row's least and greatest key
                    uint32_t least = 0xffffffffu, most = 0u;
#pragma unroll
                    for (int i = 0; i < E; ++i)
                        if (4 * (t + L * (i / 4)) < D) {
                            least = min(least, key[i]);
                            most = max(most, key[i]);
                        }
                    least = ~group_max<L>(~least);
                    most = group_max<L>(most);
                    if (trip == 0 && reach == kWalk) note();
                    const bool has_lo = fabsf(lof) < __builtin_inff(), has_hi = fabsf(hif) < __builtin_inff();
                    lo = has_lo ? key_of(lof) : least;
                    clo = has_lo ? clo : (float)(D - k);
                    hi = has_hi ? key_of(hif) : most + 1u;
                    chi = has_hi ? chi : (float)-k;
                    if (__any(most == 0xffffffffu)) {         // a not-a-number of all ones: most + 1 is no key
                        uint32_t ones = 0xffffffffu;
                        asm volatile("" : "+v"(ones));        // counted here: hoisted out of the loop, every row would pay
                        const int c = (int)count(ones) - k;
                        const bool top = open && most == 0xffffffffu, ge = c >= 0;
                        lo = top && ge ? 0xffffffffu : lo;    // hi - lo is taken modulo 2^32
                        hi = top ? (ge ? 0u : (has_hi ? hi : 0xffffffffu)) : hi;
                        chi = top && !ge && !has_hi ? (float)c : chi;
                    }
                }
                for (; __any(open); ++trip) {
                    uint32_t next = lo + ((hi - lo) >> 1);
                    if (trip & 1) {
                        const float part = (float)(hi - lo) * ((clo + 0.5f) * __builtin_amdgcn_rcpf(clo - chi + 1.0f));
                        next = lo + min(max((uint32_t)part, 1u), hi - lo - 1u);
                    }
                    cand = open ? next : cand;
                    const int c = (int)count(cand) - k;
                    uint32_t below, above;
                    neighbours(cand, &below, &above);         // the bracket's ends are keys of the row: few distinct ones, few trips
                    const bool ge = open && c >= 0, lt = open && c < 0;
                    lo = ge ? cand + above : lo;
                    clo = ge ? (float)c : clo;
                    hi = lt ? cand + below + 1u : hi;
                    chi = lt ? (float)c : chi;
                    d = open ? c : d;
                    const bool met = hi - lo <= 1u;
                    cand = open && met ? lo : cand;
                    d = open && met ? 0 : d;                  // nothing to walk: what is kept is counted below
                    open = open && !met && abs(d) > reach;
                }
                if (lost && __any(hi - lo > 1u)) {            // the distance of values near T
                    const float near = (value_of(hi) - value_of(lo)) * __builtin_amdgcn_rcpf(clo - chi);
                    g.gap = hi - lo > 1u && near < __builtin_inff() ? near : g.gap;
                    trace.lost = true;
                    if constexpr (TRACE == 1) trace.g.gap = g.gap;
                }
            }
            for (int it = 0; it < reach && __any(d != 0); ++it) {
                uint32_t below, above;
                neighbours(cand, &below, &above);
                cand += d < 0 ? below : (d > 0 ? above + 1u : 0u);
                d += d < 0 ? 1 : (d > 0 ? -1 : 0);
            }
            *at = starts(t, [&](int i) { return key[i] >= cand; }, &kept);
            open = kept != (uint32_t)k;
            *ties = __any(open);
            if (reach == 0 || !*ties) break;
        }
        if constexpr (TRACE == 2) trace.g = g;
        return cand;
    }
    // Where to begin: as if its values were normally distributed.
    __device__ __forceinline__ Guide guide(int t, int D, const FirstGuess& f) const {
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int i = 0; i < E; ++i)
            if (4 * (t + L * (i / 4)) < D) {
                s1 += v[i];
                s2 = fmaf(v[i], v[i], s2);
            }
        auto more = [](float x, auto ctrl) { return x + __uint_as_float(lane_swap<decltype(ctrl)::value>(__float_as_uint(x))); };
        auto both = [&](auto ctrl) { s1 = more(s1, ctrl); s2 = more(s2, ctrl); };
        both(std::integral_constant<int, kQuadXor1>{});
        both(std::integral_constant<int, kQuadXor2>{});
        if constexpr (L >= 8) both(std::integral_constant<int, kHalfMirror>{});
        if constexpr (L >= 16) both(std::integral_constant<int, kMirror>{});
        const float r = __builtin_amdgcn_rcpf((float)D), mean = s1 * r;
        const float sigma = __builtin_amdgcn_sqrtf(fmaxf(s2 * r - mean * mean, 0.0f)), gap = sigma * f.gap;
        const bool fine = gap < __builtin_inff() && fabsf(mean) < __builtin_inff();      // also false where it is not a number
        return Guide{fine ? fmaf(sigma, f.z, mean) : 0.0f, fine ? gap : 1.0f};
    }
    // Per slot, how many of the flags before this lane's (in the order of the columns) are set: byte s of the result.  *total: of
    // the whole row.
    template <typename F> __device__ __forceinline__ uint32_t starts(int t, F flag, uint32_t* total) const {
        uint32_t n = 0;
#pragma unroll
        for (int s = SLOTS - 1; s >= 0; --s) {
            uint32_t c = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) c += flag(4 * s + j) ? 1u : 0u;
            n = (n << 8) + c;
        }
        const uint32_t all = group_sum<L>(n);
        *total = (all & 0xffu) + (all >> 8 & 0xffu) + (all >> 16 & 0xffu) + (all >> 24);
        return group_before<L>(n, t) + (all << 8) + (all << 16) + (all << 24);     // at most 252: no byte runs over
    }
    // Of the keys equal to T only the first columns are kept, k in all: the others' keys are cleared.  Returns the threshold from
    // then on: 0, the key of one not-a-number and of what is no column, becomes 1, so that what is cleared lies below it.
    __device__ __forceinline__ uint32_t drop_ties(uint32_t T, int k, int t) {
        uint32_t above = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) above += key[i] > T ? 1u : 0u;
        const uint32_t need = (uint32_t)k - group_sum<L>(above);
        uint32_t equal;
        const uint32_t at = starts(t, [&](int i) { return key[i] == T; }, &equal), from = max(T, 1u);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            uint32_t rank = (at >> (8 * s)) & 0xffu;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool eq = key[4 * s + j] == T;
                key[4 * s + j] = eq ? (rank < need ? from : 0u) : key[4 * s + j];
                rank += eq ? 1u : 0u;
            }
        }
        return from;
    }
    // kept pairs to pairs[0 .. k) of the row; `spare`: a place of this lane's own for what is not kept
    __device__ __forceinline__ void place(uint32_t T, uint32_t at, int t, uint2* pairs, uint2* spare) const {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            uint2* to = pairs + ((at >> (8 * s)) & 0xffu);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool keep = key[4 * s + j] >= T;
                *(keep ? to : spare) = make_uint2(__float_as_uint(v[4 * s + j]), (uint32_t)(4 * (t + L * s) + j));
                to += keep ? 1 : 0;
            }
        }
    }
};

template <int L, int SLOTS, bool DUAL>
__global__ __launch_bounds__(256) void topk_groups_kernel(TopkArgs args) {
    extern __shared__ uint4 kept_keys4[];                     // per wavefront: 64 spare places, then the kept pairs of its rows
    constexpr int R = kWave / L;                              // rows per wavefront
    using Row = GroupRow<L, SLOTS>;
    int sg = 0;
    while (sg + 1 < args.n && (int)blockIdx.x >= args.s[sg + 1].blk0) ++sg;
    const TopkSeg& seg = args.s[sg];
    const float* __restrict__ X = seg.X;
    const int n = seg.n, D = args.D;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = lane & (L - 1), g = lane / L;
    uint2* const spare = reinterpret_cast<uint2*>(kept_keys4) + wave * (kWave + R * args.k_max) + lane;
    uint2* const pairs = spare - lane + kWave;
    const uint32_t stride = (uint32_t)seg.n_blocks * 4u * R;
    uint32_t row0 = ((uint32_t)(blockIdx.x - seg.blk0) * 4u + (uint32_t)wave) * R;

    float4v next[SLOTS];
    auto load = [&](uint32_t first) {                         // rows and columns past the end: clamped to valid addresses
        const float* x = X + (size_t)min(first + (uint32_t)g, (uint32_t)n - 1u) * D;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int c = 4 * (t + L * s);
            next[s] = __builtin_nontemporal_load(reinterpret_cast<const float4v*>(x + (c < D ? c : 0)));     // read once
        }
    };
    Row row;
    Trace trace{};
    auto select = [&](int k, float* __restrict__ vals, uint16_t* __restrict__ idx, const FirstGuess& guess, auto how) __attribute__((always_inline)) {
        constexpr int TRACE = decltype(how)::value;
        bool ties;
        uint32_t at, kept;
        uint32_t T = row.template threshold<TRACE>(k, t, D, guess, trace, &at, &ties);
        if (TRACE == 2 || (TRACE == 1 && trace.lost)) {
            // Taken up when it is called for, left when it leads astray itself.  Rows with equal values at T leave none: they are as
            // far from there the next time.
            const float x = value_of(T), to = trace.on ? trace.g.at + 0.25f * (x - trace.g.at) : x;
            trace.g.at = fabsf(to) < __builtin_inff() ? to : 0.0f;
            trace.on = trace.on ? !trace.lost : trace.lost && !ties;
            trace.lost = false;
        }
        if (ties) {
            T = row.drop_ties(T, k, t);
            at = row.starts(t, [&](int i) { return row.key[i] >= T; }, &kept);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // one wavefront's LDS accesses run in program order
        __builtin_amdgcn_wave_barrier();
        row.place(T, at, t, pairs + g * k, spare);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the pairs of the wavefront's rows are one stretch of the output, which starts at a multiple of four pairs
        const int total = (int)min((uint32_t)R, (uint32_t)n - row0) * k;
        const size_t base = (size_t)row0 * k;
        for (int p = 4 * lane; p < total; p += 4 * kWave) {
            const uint4 a = reinterpret_cast<const uint4*>(pairs)[p / 2], b = reinterpret_cast<const uint4*>(pairs)[p / 2 + 1];
            if (seg.wide_out && p + 4 <= total) {
                *reinterpret_cast<float4v*>(vals + base + p) =
                    float4v{__uint_as_float(a.x), __uint_as_float(a.z), __uint_as_float(b.x), __uint_as_float(b.z)};
                *reinterpret_cast<uint2*>(idx + base + p) = make_uint2(a.y | a.w << 16, b.y | b.w << 16);
            } else {
                const uint32_t vv[4] = {a.x, a.z, b.x, b.z}, cc[4] = {a.y, a.w, b.y, b.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (p + j < total) {
                        vals[base + p + j] = __uint_as_float(vv[j]);
                        idx[base + p + j] = (uint16_t)cc[j];
                    }
            }
        }
        return ties;
    };
    if (row0 >= (uint32_t)n) return;
    load(row0);
    // true: no row is left; false: the trips to come follow a trace
    auto trips = [&](auto how) __attribute__((always_inline)) {
        constexpr int TRACE = decltype(how)::value;
        for (;; row0 += stride) {
#pragma unroll
            for (int i = 0; i < Row::E; ++i) row.v[i] = next[i / 4][i & 3];
            const bool more = (uint32_t)n - row0 > stride;
            if (more) load(row0 + stride);                    // in flight while these rows are selected
            row.make_keys(t, D);
            const bool ties = select(seg.k, seg.vals, seg.idx, seg.guess, how);
            if constexpr (DUAL) {
                if (seg.vals2) {
                    if (ties) row.make_keys(t, D);
                    select(seg.k2, seg.vals2, seg.idx2, seg.guess2, how);
                }
            }
            if (!more) return true;
            if (TRACE == 1 && trace.on) break;
        }
        row0 += stride;
        return false;
    };
    // A trace takes registers (two selections have none to spare) and pays from the second trip on (16 lanes a row have one) where the
    // search is long; its loop is one of its own because the other's rows would pay for a test and two selects (2 %).
    if constexpr (!DUAL && L < 16 && SLOTS == 4) {
        if (!trips(std::integral_constant<int, 1>{})) trips(std::integral_constant<int, 2>{});
    } else {
        trips(std::integral_constant<int, 0>{});
    }
}

template <int L, int SLOTS>
static void launch_groups(const TopkArgs& a, int blocks, bool dual, hipStream_t s) {
    const size_t lds = sizeof(uint2) * 4 * (kWave + (size_t)(kWave / L) * a.k_max);
    if (dual) hipLaunchKernelGGL((topk_groups_kernel<L, SLOTS, true>), dim3((unsigned)blocks), dim3(256), lds, s, a);
    else hipLaunchKernelGGL((topk_groups_kernel<L, SLOTS, false>), dim3((unsigned)blocks), dim3(256), lds, s, a);
}
// Few rows (less than kFewRows in all) are spread over more lanes: fewer elements per lane shorten the one chain a wavefront
// goes through.  Rows a wavefront takes at a time:
static int group_rows(int D, bool few) { return few ? 4 : (D <= 64 ? 16 : 8); }

template <int EPL>
static void launch_epl(const TopkArgs& a, int blocks, bool dual, int ranked_k, hipStream_t s) {
    if (ranked_k)
        hipLaunchKernelGGL((topk_rows_kernel<EPL, false, true>), dim3((unsigned)blocks), dim3(256),
                           sizeof(uint4) * 4 * (size_t)((ranked_k + 3) / 4), s, a);
    else if (dual)
        hipLaunchKernelGGL((topk_rows_kernel<EPL, true, false>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((topk_rows_kernel<EPL, false, false>), dim3((unsigned)blocks), dim3(256), 0, s, a);
}

static int launch_any(const TopkJob* jobs, int n, int D, bool ranked, hipStream_t s) {
    // Whole float4s of rows of up to 128 columns: several rows per wavefront.  Wider rows gain less by it (250 000 x 256, k = 64:
    // 86 -> 74 us on normal data, 100 -> 125 on skewed data), and the rank order is found per wavefront.
    bool groups = !ranked && D <= 128 && D % 4 == 0;
    int64_t rows = 0;
    for (int i = 0; i < n; ++i) {
        groups = groups && aligned(jobs[i].X, 16);
        rows += jobs[i].n;
    }
    const bool few = rows < kFewRows;
    for (int i = 0; i < n;) {
        TopkArgs a{};
        a.D = D;
        int blocks = 0;
        bool dual = false;
        for (; i < n && a.n < kTopkSegs; ++i) {
            const TopkJob& j = jobs[i];
            if (j.n == 0) continue;
            int64_t b;
            if (groups) {
                b = (j.n + 4 * group_rows(D, few) - 1) / (4 * group_rows(D, few));
                if (b > kGroupBlocks) b = kGroupBlocks;
            } else {
                // Each wavefront strides over rows with four of them in flight, so it wants at least four rows (a wavefront
                // with one row pays the whole load latency for it: 20 000 rows took 15 us on 4096 workgroups, 9 us on 1250);
                // beyond 8192 workgroups (four rounds of 8 waves per SIMD) nothing is gained.  Measured on 20 k ... 1.2 M rows.
                b = (j.n + 15) / 16;
                if (b > 8192) b = 8192;
            }
            a.s[a.n++] = TopkSeg{j.X, j.vals, j.vals2, j.idx, j.idx2, (int)j.n, j.k, j.k2, blocks, (int)b,
                                 aligned(j.vals, 16) && aligned(j.idx, 8) && aligned(j.vals2, 16) && aligned(j.idx2, 8) ? 1 : 0,
                                 groups ? first_guess(D, j.k) : FirstGuess{}, groups && j.vals2 ? first_guess(D, j.k2) : FirstGuess{}};
            if (j.k > a.k_max) a.k_max = j.k;
            if (j.vals2 && j.k2 > a.k_max) a.k_max = j.k2;
            blocks += (int)b;
            dual = dual || j.vals2;
        }
        if (a.n == 0) break;
        if (groups) {
            if (few && D <= 64) launch_groups<16, 1>(a, blocks, dual, s);
            else if (few && D <= 128) launch_groups<16, 2>(a, blocks, dual, s);
            else if (D <= 32) launch_groups<4, 2>(a, blocks, dual, s);
            else if (D <= 64) launch_groups<4, 4>(a, blocks, dual, s);
            else if (D <= 96) launch_groups<8, 3>(a, blocks, dual, s);
            else launch_groups<8, 4>(a, blocks, dual, s);
            continue;
        }
        const int rk = ranked ? a.s[0].k : 0;
        if (D <= 64) launch_epl<1>(a, blocks, dual, rk, s);
        else if (D <= 128) launch_epl<2>(a, blocks, dual, rk, s);
        else if (D <= 256) launch_epl<4>(a, blocks, dual, rk, s);
        else if (D <= 512) launch_epl<8>(a, blocks, dual, rk, s);
        else launch_epl<16>(a, blocks, dual, rk, s);
    }
    DRC_HIP(hipGetLastError());
    return DR_OK;
}

int launch_topks(const TopkJob* jobs, int n, int D, hipStream_t s) { return launch_any(jobs, n, D, false, s); }

int launch_topk(const float* X, int64_t n, int D, int k, float* vals, uint16_t* idx, hipStream_t s) {
    const TopkJob j{X, n, k, vals, idx, 0, nullptr, nullptr};
    return launch_any(&j, 1, D, false, s);
}

int launch_topk_ranked(const float* X, int64_t n, int D, int k, float* vals, uint16_t* idx, hipStream_t s) {
    const TopkJob j{X, n, k, vals, idx, 0, nullptr, nullptr};
    return launch_any(&j, 1, D, true, s);
}

}  // namespace drc
