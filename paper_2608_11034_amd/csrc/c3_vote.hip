// Consensus kernels of C3 for gfx950: the decision step of Algorithm 1.
//
// Which kernel decides a unit depends on the group size R:
//   R <= 32   one thread per unit, the R values in registers (128-bit row
//             loads when replicas are adjacent), deciding with the per-unit
//             functions of c3_vote_row.h (fp64 statistics up to R = 16);
//   above     exact: one wave per unit, lane l holding replicas l, l + 64,
//             ..., candidate values broadcast by readlane, bitmap word s one
//             ballot; statistical: sixteen lanes per unit, which sort the
//             unit's values once.
// On 1M-unit rows the wave's exact vote was up to 7.6x (R = 64) faster than
// lane-per-replica counting.
//
// EXACT (Sec. 5.3): a strict majority exists iff some value is held by more
// than R / 2 replicas; those are the majority, the bitmap marks the others
// and the majority index is the lowest majority replica.
//
// STATISTICAL (Sec. 5.4), in fp64: order statistics of the finite values in
// the stable (value, then replica index) order give the median, the median
// absolute deviation, the type-7 quartiles and the range, in the fallback
// order MAD -> IQR / 2 -> range / n_finite.  Non-finite values are outliers
// and take no part in m or d.  No floating-point contraction is allowed in
// this file (the host compiles it with -ffp-contract=off), so the decision
// rounds exactly as the plain definition does.
#include "c3_device.h"
#include "c3_internal.h"
#include "c3_vote_row.h"

namespace c3 {

constexpr int kVoteThreads = 256;

// ---------------------------------------------------------------------------
// Small groups (R <= 32): one thread per unit with the R values in registers,
// so the whole decision is register arithmetic.  NMAX is R rounded up to a
// power of two; slots past R are padding that never takes part.
// ---------------------------------------------------------------------------
template <int NMAX>
__global__ void __launch_bounds__(kVoteThreads) exact_vote_small_kernel(
    const char* __restrict__ ev, int kind, int64_t rstride, int64_t ustride, int R, int64_t n_units,
    bool dense, uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
    int32_t* __restrict__ majority_idx) {
    const int64_t u = (int64_t)blockIdx.x * kVoteThreads + threadIdx.x;
    if (u >= n_units) return;
    uint64_t e[NMAX];
    load_row_bits<NMAX>(ev + u * ustride, kind, rstride, R, dense, e);
    const UnitVote v = exact_vote_row<NMAX>(e, R);
    status[u] = v.status;
    bitmap[u] = v.bitmap;
    majority_idx[u] = v.majority;
}

template <int NMAX, int KIND>
__global__ void __launch_bounds__(kVoteThreads) statistical_vote_small_kernel(
    const char* __restrict__ ev, int kind, int64_t rstride, int64_t ustride, int R, int64_t n_units,
    bool dense, double kappa, uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
    int32_t* __restrict__ majority_idx) {
    const int64_t u = (int64_t)blockIdx.x * kVoteThreads + threadIdx.x;
    if (u >= n_units) return;
    uint64_t bits[NMAX];
    load_row_bits<NMAX>(ev + u * ustride, kind, rstride, R, dense, bits);
    const UnitVote v = statistical_vote_row<NMAX, KIND>(bits, R, kappa);
    status[u] = v.status;
    bitmap[u] = v.bitmap;
    majority_idx[u] = v.majority;
}

// ---------------------------------------------------------------------------
// Wave per unit (every group above 32 replicas).  Lane l
// holds the values of replicas l, l + 64, l + 128 and l + 192 (NS =
// ceil(R / 64) slots; slot s holds replica 64 s + l), so bitmap word s is the
// ballot of slot s.  The exact vote broadcasts candidate values by readlane
// at a wave-uniform index; the statistical vote sorts the wave's values.
// ---------------------------------------------------------------------------
constexpr int kWideUnitsPerBlock = kVoteThreads / 64;

// Value of replica j (wave-uniform) from the slot registers.
template <int NS>
__device__ inline uint64_t wide_value(const uint64_t (&e)[NS], int j) {
    uint64_t v = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s == (j >> 6)) v = readlane_u64(e[s], j & 63);
    return v;
}

template <int NS>
__device__ inline void wide_write(int64_t u, uint8_t st, const uint64_t (&b)[NS], int32_t mj,
                                  uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
                                  int32_t* __restrict__ majority_idx) {
    if ((threadIdx.x & 63) != 0) return;
    status[u] = st;
    majority_idx[u] = mj;
#pragma unroll
    for (int s = 0; s < NS; ++s) bitmap[u * NS + s] = b[s];
}

// EXACT: a strict majority has more than R / 2 members, so one of replicas
// 0 .. floor(R / 2) holds it.  Candidate values are tried from the lowest
// such replica not yet covered, each with one broadcast and NS ballots; a
// failed value marks every replica holding it, so each distinct value is
// tried once.  The usual unit (replica 0 in the majority) needs one try, a
// two-way split two.  A unit whose candidates all fail has no strict
// majority.
template <int NS>
__global__ void __launch_bounds__(kVoteThreads) exact_vote_wide_kernel(
    const char* __restrict__ ev, int kind, int64_t rstride, int64_t ustride, int R, int64_t n_units,
    uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap, int32_t* __restrict__ majority_idx) {
    const int lane = threadIdx.x & 63;
    const int64_t u = (int64_t)blockIdx.x * kWideUnitsPerBlock + (threadIdx.x >> 6);
    if (u >= n_units) return;  // the whole wave leaves together
    uint64_t e[NS];
    bool valid[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int r = 64 * s + lane;
        valid[s] = r < R;
        e[s] = valid[s] ? load_ev_bits(ev + u * ustride + (int64_t)r * rstride, kind) : 0ull;
    }
    uint64_t cand = 0;
    int cnt = 0;
    bool tried[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) tried[s] = false;
    int j = 0;
    while (true) {  // at most floor(R / 2) + 1 rounds: each covers replica j
        cand = wide_value<NS>(e, j);
        cnt = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bool eq = valid[s] && e[s] == cand;
            cnt += __builtin_popcountll(ballot64(eq));
            tried[s] = tried[s] || eq;
        }
        if (2 * cnt > R) break;
        j = -1;
#pragma unroll
        for (int s = NS - 1; s >= 0; --s) {
            const uint64_t b = ballot64(!tried[s] && 64 * s + lane <= R / 2);
            if (b) j = 64 * s + __builtin_ctzll(b);
        }
        if (j < 0) break;
    }
    uint64_t ob[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) ob[s] = 0;
    if (2 * cnt <= R) {
        wide_write<NS>(u, C3_INCONCLUSIVE, ob, -1, status, bitmap, majority_idx);
        return;
    }
    int mj = -1;
    bool any = false;
#pragma unroll
    for (int s = NS - 1; s >= 0; --s) {
        const uint64_t mb = ballot64(valid[s] && e[s] == cand);
        ob[s] = ballot64(valid[s] && e[s] != cand);
        if (mb) mj = 64 * s + __builtin_ctzll(mb);
        any = any || ob[s] != 0;
    }
    wide_write<NS>(u, any ? C3_ATTRIBUTED : C3_AGREE, ob, mj, status, bitmap, majority_idx);
}

// STATISTICAL over more than 32 replicas (fp64: 16): sixteen lanes decide a
// unit, four units a wave.
//
// Lane l of the sixteen loads replicas l, l + 16, ... (NL of them, so a load
// reads four runs of sixteen adjacent values), the group sorts the finite
// values once and every order statistic is read off the sorted copy in LDS.
// Sorted position p = NL l + i is register i of lane l (excluded values as
// +inf): the network's short distances, the most frequent ones, are
// comparators between a lane's own registers, one instruction per value and
// stage, and only the distances between lanes, at most 15, cost a DPP move and
// a select.  The network is
// the bitonic sorter in its one-direction form: merging blocks of B lanes,
// (lane, i) first meets (lane ^ (B - 1), NL - 1 - i), the reversed other half,
// then lane ^ B / 4 .. lane ^ 1, and then a lane's own bitonic run is sorted.
// Values only: equal values are interchangeable, and the lower-median replica
// is found afterwards by counting.
//
// VALU-bound.  262,144 units, us per call, against one wave per unit with
// R / 64 values a lane and order statistics by readlane:
//   R          33     64    128    192    256
//   fp32     82->42 92->45 179->73 265->105 288->139
//   fp64     91->53 102->55 198->99 314->156 335->221

template <int M>
__device__ __forceinline__ uint32_t row_lane_u32(uint32_t v) {   // lane ^ M within a row of 16
    const int iv = (int)v;
    if constexpr (M == 3) return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x1B, 0xF, 0xF, false);
    else if constexpr (M == 7) return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x141, 0xF, 0xF, false);
    else if constexpr (M == 15) return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x140, 0xF, 0xF, false);
    else return row_xor_u32<M>(v);
}
template <int M>
__device__ __forceinline__ float row_lane(float v) {
    return __uint_as_float(row_lane_u32<M>(__float_as_uint(v)));
}
template <int M>
__device__ __forceinline__ double row_lane(double v) {
    const uint64_t b = bits_of(v);
    const uint64_t lo = row_lane_u32<M>((uint32_t)b), hi = row_lane_u32<M>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((hi << 32) | lo));
}

// Between lanes: the lane in the lower half of the pair keeps the smaller
// value.  The median of a, b and -inf is their minimum, of a, b and +inf
// their maximum, so one instruction serves both halves in fp32.
struct KeepF32 {
    float c;
    __device__ explicit KeepF32(bool upper) : c(upper ? __builtin_huge_valf() : -__builtin_huge_valf()) {}
    __device__ __forceinline__ float operator()(float a, float b) const {
        return __builtin_amdgcn_fmed3f(a, b, c);
    }
};
struct KeepF64 {
    bool upper;
    __device__ explicit KeepF64(bool u) : upper(u) {}
    __device__ __forceinline__ double operator()(double a, double b) const {
        return ((b < a) != upper) ? b : a;
    }
};

// Plain min and max between a lane's own registers.  The builtins rather than
// inline assembly: their results feed DPP moves, whose wait states the
// compiler places only after instructions that it knows.
__device__ __forceinline__ void order_pair(float& a, float& b) {
    const float lo = __builtin_fminf(a, b), hi = __builtin_fmaxf(a, b);
    a = lo;
    b = hi;
}
__device__ __forceinline__ void order_pair(double& a, double& b) {
    const double lo = __builtin_fmin(a, b), hi = __builtin_fmax(a, b);
    a = lo;
    b = hi;
}
template <typename V>
__device__ __forceinline__ void order_three(V& a, V& b, V& c) {
    order_pair(a, b);
    order_pair(b, c);
    order_pair(a, b);
}

// Sorts registers [at, at + N) that hold a bitonic run (half-cleaners work on
// any even length, so twelve go 6, 3 and then threes).
template <int N, int NL, typename V>
__device__ __forceinline__ void sort_run(V (&k)[NL], int at) {
    if constexpr (N == 3) {
        order_three(k[at], k[at + 1], k[at + 2]);
    } else if constexpr (N >= 2) {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) order_pair(k[at + i], k[at + i + N / 2]);
        sort_run<N / 2>(k, at);
        sort_run<N / 2>(k, at + N / 2);
    }
}
// Sorts registers [at, at + N): halves, then the reversed merge.  (Batcher's
// network would save 17 of 80 comparators at 16, 2% of the whole sort.)
template <int N, int NL, typename V>
__device__ __forceinline__ void sort_lane(V (&k)[NL], int at) {
    if constexpr (N == 3) {
        order_three(k[at], k[at + 1], k[at + 2]);
    } else if constexpr (N >= 2) {
        sort_lane<N / 2>(k, at);
        sort_lane<N / 2>(k, at + N / 2);
#pragma unroll
        for (int i = 0; i < N / 2; ++i) order_pair(k[at + i], k[at + N - 1 - i]);
        sort_run<N / 2>(k, at);
        sort_run<N / 2>(k, at + N / 2);
    }
}
template <int M, int NL, typename V>
__device__ __forceinline__ void sort_halves(V (&k)[NL], int lane) {
    using Keep = typename std::conditional<sizeof(V) == 4, KeepF32, KeepF64>::type;
    if constexpr (M >= 1) {
        const Keep keep((lane & M) != 0);
#pragma unroll
        for (int i = 0; i < NL; ++i) k[i] = keep(k[i], row_lane<M>(k[i]));
        sort_halves<M / 2>(k, lane);
    }
}
template <int B, int NL, typename V>
__device__ __forceinline__ void sort_merge(V (&k)[NL], int lane) {
    using Keep = typename std::conditional<sizeof(V) == 4, KeepF32, KeepF64>::type;
    if constexpr (B <= 16) {
        const Keep keep((lane & (B / 2)) != 0);
        V o[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) o[i] = row_lane<B - 1>(k[NL - 1 - i]);
#pragma unroll
        for (int i = 0; i < NL; ++i) k[i] = keep(k[i], o[i]);
        sort_halves<B / 4>(k, lane);
        sort_run<NL>(k, 0);
        sort_merge<2 * B>(k, lane);
    }
}

__device__ __forceinline__ uint32_t row_sum_u32(uint32_t v) {
    v += row_xor_u32<8>(v);
    v += row_xor_u32<4>(v);
    v += row_xor_u32<2>(v);
    return v + row_xor_u32<1>(v);
}
__device__ __forceinline__ uint32_t row_min_u32(uint32_t v) {
    v = min(v, row_xor_u32<8>(v));
    v = min(v, row_xor_u32<4>(v));
    v = min(v, row_xor_u32<2>(v));
    return min(v, row_xor_u32<1>(v));
}

// The lowest R that takes NL registers a lane.
constexpr int stat_least(int nl) { return nl == 2 ? 17 : nl == 4 ? 33 : nl == 8 ? 65 : nl == 12 ? 129 : 193; }
constexpr int kStatUnits = kVoteThreads / 16;      // units per workgroup

// One group's decision: NS bitmap words, whether any bit is set, the majority
// replica, and whether the unit is conclusive.
template <int NL>
struct GroupVote {
    static constexpr int NS = (NL + 3) / 4;
    uint64_t B[NS];
    int mj;
    bool ok, any;
};

template <int NL>
__device__ __forceinline__ void write_group(const GroupVote<NL>& v, int64_t u, int l,
                                            uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
                                            int32_t* __restrict__ majority_idx) {
    constexpr int NS = GroupVote<NL>::NS;
    if (l == 0 && status != nullptr) {
        status[u] = !v.ok ? (uint8_t)C3_INCONCLUSIVE : v.any ? (uint8_t)C3_ATTRIBUTED : (uint8_t)C3_AGREE;
        majority_idx[u] = v.ok ? v.mj : -1;
    }
#pragma unroll
    for (int w = 0; w < NS; ++w)
        if (l == w) bitmap[u * NS + w] = v.B[w];
}

// Whether replica 16 j + l exists, decided at compile time where NL says so.
template <int NL>
__device__ __forceinline__ bool group_valid(int j, int l, int R) {
    return 16 * (j + 1) <= stat_least(NL) || 16 * j + l < R;
}

// The statistical decision of a unit whose sixteen lanes hold x (replica 16 j
// + l in x[j], +inf where excluded; bit j of `bad`: a replica that is not
// finite); s: 16 NL slots of LDS of their own.
template <int NL, typename V>
__device__ __forceinline__ GroupVote<NL> stat_group(const V (&x)[NL], uint32_t bad, int R, double kappa,
                                                    V* s, int l, int q4) {
    constexpr int NS = GroupVote<NL>::NS;
    const V inf = (V)__builtin_huge_val();
    V k[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) k[j] = x[j];
    int nf = R;
    const bool some_bad = ballot64(bad != 0u) != 0ull;
    if (some_bad) nf -= (int)row_sum_u32((uint32_t)__builtin_popcount(bad));
    const bool ok = 2 * nf > R;                     // finite values are a strict majority
    const int n = nf > 1 ? nf : 1;
    sort_lane<NL>(k, 0);
    sort_merge<2>(k, l);
#pragma unroll
    for (int i = 0; i < NL; ++i) s[NL * l + i] = k[i];
    wave_lds_sync();
    auto S = [&](int p) { return (double)s[p]; };

    const int pm = (n - 1) / 2;
    const V target = s[pm];                         // the lower median
    const double a0 = (double)target, b0 = S(n / 2);
    const double m = (n & 1) ? a0 : (a0 + b0) * 0.5;
    // values below the lower median, its holders, and the first holder
    uint32_t cnt = 0, holder = 0xFFFFu;
#pragma unroll
    for (int j = NL - 1; j >= 0; --j) {
        cnt += (uint32_t)(x[j] < target);
        cnt += x[j] == target ? 0x10000u : 0u;
        holder = x[j] == target ? (uint32_t)(16 * j + l) : holder;
    }
    cnt = row_sum_u32(cnt);
    const int less = (int)(cnt & 0xFFFFu), same = (int)(cnt >> 16);
    int mj = (int)row_min_u32(holder);
    if (ballot64(same > 1) != 0ull) {
        // ties: position pm of the stable (value, replica) order is holder
        // pm - less, counted by replica index
        int want = pm - less;
        mj = -1;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            uint32_t eq = (uint32_t)(ballot64(x[j] == target) >> (16 * q4)) & 0xFFFFu;
            const int c = __builtin_popcount(eq);
            if (mj < 0 && want < c) {
                for (int w = 0; w < want; ++w) eq &= eq - 1u;
                mj = 16 * j + __builtin_ctz(eq | 0x10000u);
            }
            want -= c;
        }
    }
    // The values below m: no value lies between the middle two, so they are
    // those up to the lower middle one, or, where that equals m, those below
    // it.  (The last two cases only where the sum of the middle two overflows.)
    const int split = a0 < m ? (b0 < m ? n : pm + 1) : (a0 > m ? 0 : less);

    // Median of |s - m| over the n sorted values without sorting the
    // deviations: the `split` values below m give m - s[split - 1 - i], the
    // others s[split + i] - m, two ascending runs (each deviation rounds as
    // |s - m| does, since rounding is symmetric).  How many of the pm + 1
    // smallest come from the first run is found by two rounds of sixteen
    // probes.
    const int nl = split, nh = n - split;
    auto at = [&](int p) { return S(p < 0 ? 0 : p < 16 * NL ? p : 16 * NL - 1); };
    auto L = [&](int i) { return m - at(split - 1 - i); };
    auto H = [&](int i) { return at(split + i) - m; };
    int lo = pm + 1 - nh > 0 ? pm + 1 - nh : 0;
    int hi = pm + 1 < nl ? pm + 1 : nl;
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const int step = hi > lo ? (hi - lo + 15) >> 4 : 0;
        const int p = lo + l * step;
        const bool from_l = p < hi && L(p) < H(pm - p);
        const int c = __builtin_popcount((uint32_t)(ballot64(from_l) >> (16 * q4)) & 0xFFFFu);
        const int last = lo + (c - 1) * step;
        hi = c > 0 ? (hi < last + step ? hi : last + step) : lo;
        lo = c > 0 ? last + 1 : lo;
    }
    double d;
    {
        const double ninf = -__builtin_huge_val(), pinf = __builtin_huge_val();
        const double a = fmax(lo > 0 ? L(lo - 1) : ninf, pm - lo >= 0 ? H(pm - lo) : ninf);
        const double b = fmin(lo < nl ? L(lo) : pinf, pm + 1 - lo < nh ? H(pm + 1 - lo) : pinf);
        d = (n & 1) ? a : (a + b) * 0.5;
    }
    const double s0 = S(0), s1 = S(n - 1);
    if (d == 0.0) {
        // Hyndman-Fan type 7: h = (n - 1) p; Q = s[floor h] + frac(h) (s[floor h + 1] - s[floor h])
        auto quantile7 = [&](double p) {
            const double h = (double)(n - 1) * p;
            const double fl = floor(h);
            const int at_lo = (int)fl;
            const double frac = h - fl;
            if (at_lo + 1 >= n) return s1;
            const double a = S(at_lo);
            const double diff = S(at_lo + 1) - a;
            const double prod = frac * diff;
            return a + prod;
        };
        d = (quantile7(0.75) - quantile7(0.25)) * 0.5;
        if (d == 0.0) d = (s1 - s0) / (double)n;
    }
    const double thr = kappa * d;
    // the largest deviation is that of an end: the usual unit flags nothing
    const bool far = ok && d != 0.0 && fmax(fabs(s0 - m), fabs(s1 - m)) > thr;
    GroupVote<NL> v;
    uint64_t (&B)[NS] = v.B;
#pragma unroll
    for (int w = 0; w < NS; ++w) B[w] = 0;
    bool any = false;
    if (ballot64(far || bad != 0u) != 0ull) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            // a non-finite value is an outlier
            const bool flag = ok && (((bad >> j) & 1u) != 0u ||
                                     (far && x[j] < inf && fabs((double)x[j] - m) > thr));
            const uint32_t bits = (uint32_t)(ballot64(flag) >> (16 * q4)) & 0xFFFFu;
            B[j >> 2] |= (uint64_t)bits << (16 * (j & 3));
            any = any || bits != 0u;
        }
    }
    v.mj = mj;
    v.ok = ok;
    v.any = any;
    return v;
}

// `left` copies of cand, the rest of a lane's values paired off, meets the
// other lane's.
template <int M>
__device__ __forceinline__ void majority_level(uint64_t& cand, uint32_t& left) {
    const uint64_t c = row_xor_u64<M>(cand);
    const uint32_t n = row_xor_u32<M>(left);
    const bool same = c == cand, mine = left >= n;
    cand = same || mine ? cand : c;
    left = same ? left + n : mine ? left - n : n - left;
}

// The exact decision of a unit whose sixteen lanes hold the bits e (replica
// 16 j + l in e[j]).  The usual unit agrees with replica 0.  Otherwise pairs of
// different values are struck out (Boyer and Moore's majority vote), in each
// lane and then wherever lanes meet; a strict majority outlasts any such
// pairing, so one candidate is left to count, whatever the values are.  128
// groups over 512 iterations, us per call with none, 1% and all of the rows
// split in two halves: 32 ranks, fp64 times 16.2, 16.3, 18.3; 64 ranks, fp32
// 18.2, 18.6, 21.2.  Trying replicas 0 .. R / 2 in turn, the rest of the wave
// waiting: 16.3, 18.9, 26.5 and 18.3, 25.1, 40.0.
template <int NL>
__device__ __forceinline__ GroupVote<NL> exact_group(const uint64_t (&e)[NL], int R, int l, int q4) {
    constexpr int NS = GroupVote<NL>::NS;
    GroupVote<NL> v;
#pragma unroll
    for (int w = 0; w < NS; ++w) v.B[w] = 0;
    v.mj = 0;
    v.ok = true;
    v.any = false;
    auto from_lane = [&](uint64_t x, int src) { return shfl_u64(x, 16 * q4 + src); };
    uint64_t cand = from_lane(e[0], 0);
    bool differs = false;
#pragma unroll
    for (int j = 0; j < NL; ++j) differs = differs || (group_valid<NL>(j, l, R) && e[j] != cand);
    if (ballot64(differs) == 0ull) return v;
    auto holders = [&](uint64_t c) {
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < NL; ++j) n += (uint32_t)(group_valid<NL>(j, l, R) && e[j] == c);
        return (int)row_sum_u32(n);
    };
    uint32_t left = 0;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const bool valid = group_valid<NL>(j, l, R), first = left == 0u;
        const bool same = first || e[j] == cand;
        cand = valid && first ? e[j] : cand;
        left = !valid ? left : same ? left + 1u : left - 1u;
    }
    majority_level<8>(cand, left);
    majority_level<4>(cand, left);
    majority_level<2>(cand, left);
    majority_level<1>(cand, left);
    cand = from_lane(cand, 0);              // (lanes may end apart where there is no majority)
    const bool found = 2 * holders(cand) > R;
    v.ok = found;
    uint32_t lowest = 0xFFFFu;
#pragma unroll
    for (int j = NL - 1; j >= 0; --j) {
        const bool valid = group_valid<NL>(j, l, R), eq = e[j] == cand;
        lowest = valid && eq ? (uint32_t)(16 * j + l) : lowest;
        const uint32_t bits = (uint32_t)(ballot64(found && valid && !eq) >> (16 * q4)) & 0xFFFFu;
        v.B[j >> 2] |= (uint64_t)bits << (16 * (j & 3));
        v.any = v.any || bits != 0u;
    }
    v.mj = (int)row_min_u32(lowest);
    return v;
}

// x[j] of a unit's row, excluded values as +inf, and which are not finite.
template <int NL, typename V>
__device__ __forceinline__ uint32_t load_times(const char* row, int64_t rstride, int l, int R,
                                               V (&x)[NL]) {
    const V inf = (V)__builtin_huge_val();
    uint32_t bad = 0;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const bool valid = group_valid<NL>(j, l, R);
        x[j] = *reinterpret_cast<const V*>(row + (int64_t)(valid ? 16 * j + l : 0) * rstride);
    }
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const bool valid = group_valid<NL>(j, l, R), fin = __builtin_isfinite(x[j]);
        bad |= (uint32_t)(valid && !fin) << j;
        x[j] = valid && fin ? x[j] : inf;
    }
    return bad;
}

template <int NL, int KIND>
__global__ void __launch_bounds__(kVoteThreads) statistical_vote_wide_kernel(
    const char* __restrict__ ev, int64_t rstride, int64_t ustride, int R, int64_t n_units,
    double kappa, uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
    int32_t* __restrict__ majority_idx) {
    // fp32 evidence is ordered and compared in fp32 (the widening to fp64 is
    // exact and monotonic); every arithmetic step is fp64
    using V = typename std::conditional<KIND == C3_EV_F32, float, double>::type;
    constexpr int kPad = 16 / (int)sizeof(V);       // rows start on different LDS banks
    __shared__ __align__(16) V sorted[kStatUnits][16 * NL + kPad];
    const int lane = threadIdx.x & 63, l = lane & 15, q4 = lane >> 4;
    const int slot = threadIdx.x >> 4;
    const int64_t u = (int64_t)blockIdx.x * kStatUnits + slot;
    // whole waves past the end leave; lanes of a wave that is partly past it
    // decide the last unit again and write nothing
    if ((int64_t)blockIdx.x * kStatUnits + (threadIdx.x >> 6) * 4 >= n_units) return;
    const bool live = u < n_units;
    V x[NL];
    const uint32_t bad = load_times<NL>(ev + (live ? u : n_units - 1) * ustride, rstride, l, R, x);
    const GroupVote<NL> v = stat_group<NL>(x, bad, R, kappa, sorted[slot], l, q4);
    if (live) write_group<NL>(v, u, l, status, bitmap, majority_idx);
}

// Both votes of the timing consensus of wide groups: the fingerprint row and
// the step-time row of a unit are loaded together by the same sixteen lanes.
// Status and majority of a kind are written only when asked for (status not
// null); the bitmaps always, for the confirmation.
template <int NL, int KIND>
__global__ void __launch_bounds__(kVoteThreads) timing_votes_wide_kernel(
    const char* __restrict__ fp, const char* __restrict__ tp, int R, int64_t n_units, double kappa,
    uint8_t* __restrict__ f_status, uint64_t* __restrict__ f_bitmap, int32_t* __restrict__ f_majority,
    uint8_t* __restrict__ t_status, uint64_t* __restrict__ t_bitmap, int32_t* __restrict__ t_majority) {
    using V = typename std::conditional<KIND == C3_EV_F32, float, double>::type;
    constexpr int kPad = 16 / (int)sizeof(V);
    __shared__ __align__(16) V sorted[kStatUnits][16 * NL + kPad];
    const int lane = threadIdx.x & 63, l = lane & 15, q4 = lane >> 4;
    const int slot = threadIdx.x >> 4;
    const int64_t u = (int64_t)blockIdx.x * kStatUnits + slot;
    if ((int64_t)blockIdx.x * kStatUnits + (threadIdx.x >> 6) * 4 >= n_units) return;
    const bool live = u < n_units;
    const int64_t first = (live ? u : n_units - 1) * R;      // of the unit's values
    uint64_t e[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j)
        e[j] = reinterpret_cast<const uint64_t*>(fp)[first + (group_valid<NL>(j, l, R) ? 16 * j + l : 0)];
    V x[NL];
    const uint32_t bad = load_times<NL>(tp + first * (int64_t)sizeof(V), (int64_t)sizeof(V), l, R, x);
    const GroupVote<NL> ev = exact_group<NL>(e, R, l, q4);
    const GroupVote<NL> tv = stat_group<NL>(x, bad, R, kappa, sorted[slot], l, q4);
    if (!live) return;
    write_group<NL>(ev, u, l, f_status, f_bitmap, f_majority);
    write_group<NL>(tv, u, l, t_status, t_bitmap, t_majority);
}

hipError_t launch_timing_votes_wide(const uint64_t* fp, const void* times, int time_kind, int R,
                                    int64_t n_units, double kappa, uint8_t* f_status,
                                    uint64_t* f_bitmap, int32_t* f_majority, uint8_t* t_status,
                                    uint64_t* t_bitmap, int32_t* t_majority, hipStream_t stream) {
    if (n_units <= 0) return hipSuccess;
    const int64_t blocks = (n_units + kStatUnits - 1) / kStatUnits;
    if (n_units > kGroupMaxUnits || R < stat_least(2) || R > 64) return hipErrorInvalidValue;
    const char* f = reinterpret_cast<const char*>(fp);
    const char* t = static_cast<const char*>(times);
    auto launch = [&](auto nl, auto kind) {
        hipLaunchKernelGGL((timing_votes_wide_kernel<decltype(nl)::value, decltype(kind)::value>),
                           dim3((unsigned)blocks), dim3(kVoteThreads), 0, stream, f, t, R, n_units,
                           kappa, f_status, f_bitmap, f_majority, t_status, t_bitmap, t_majority);
    };
    using F32 = std::integral_constant<int, C3_EV_F32>;
    using F64 = std::integral_constant<int, C3_EV_F64>;
    if (R <= 32)
        time_kind == C3_EV_F32 ? launch(std::integral_constant<int, 2>{}, F32{})
                               : launch(std::integral_constant<int, 2>{}, F64{});
    else
        time_kind == C3_EV_F32 ? launch(std::integral_constant<int, 4>{}, F32{})
                               : launch(std::integral_constant<int, 4>{}, F64{});
    return hipGetLastError();
}

template <int NS>
static void launch_exact_wide(const char* e, int kind, int64_t rstride, int64_t ustride, int R,
                              int64_t n_units, uint8_t* status, uint64_t* bitmap,
                              int32_t* majority_idx, hipStream_t stream, unsigned blocks) {
    hipLaunchKernelGGL(exact_vote_wide_kernel<NS>, dim3(blocks), dim3(kVoteThreads), 0, stream, e,
                       kind, rstride, ustride, R, n_units, status, bitmap, majority_idx);
}

template <int NL>
static hipError_t launch_stat(const char* e, int kind, int64_t rstride, int64_t ustride, int R,
                              int64_t n_units, double kappa, uint8_t* status, uint64_t* bitmap,
                              int32_t* majority_idx, hipStream_t stream) {
    const int64_t blocks = (n_units + kStatUnits - 1) / kStatUnits;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (kind == C3_EV_F32)
        hipLaunchKernelGGL((statistical_vote_wide_kernel<NL, C3_EV_F32>), dim3((unsigned)blocks),
                           dim3(kVoteThreads), 0, stream, e, rstride, ustride, R, n_units, kappa,
                           status, bitmap, majority_idx);
    else
        hipLaunchKernelGGL((statistical_vote_wide_kernel<NL, C3_EV_F64>), dim3((unsigned)blocks),
                           dim3(kVoteThreads), 0, stream, e, rstride, ustride, R, n_units, kappa,
                           status, bitmap, majority_idx);
    return hipGetLastError();
}

template <int NMAX>
static void launch_small(const char* ev, int kind, int64_t rstride, int64_t ustride, int R,
                         int64_t n_units, int mode, double kappa, uint8_t* status, uint64_t* bitmap,
                         int32_t* majority_idx, hipStream_t stream, unsigned blocks) {
    const int64_t vsize = (kind == C3_EV_U64 || kind == C3_EV_F64) ? 8 : 4;
    const bool dense = rstride == vsize && ((int64_t)R * vsize) % 16 == 0 && ustride % 16 == 0 &&
                       ((uintptr_t)ev & 15) == 0;
    if (mode == C3_EXACT)
        hipLaunchKernelGGL(exact_vote_small_kernel<NMAX>, dim3(blocks), dim3(kVoteThreads), 0, stream,
                           ev, kind, rstride, ustride, R, n_units, dense, status, bitmap,
                           majority_idx);
    else if (kind == C3_EV_F32)
        hipLaunchKernelGGL((statistical_vote_small_kernel<NMAX, C3_EV_F32>), dim3(blocks),
                           dim3(kVoteThreads), 0, stream, ev, kind, rstride, ustride, R, n_units,
                           dense, kappa, status, bitmap, majority_idx);
    else
        hipLaunchKernelGGL((statistical_vote_small_kernel<NMAX, C3_EV_F64>), dim3(blocks),
                           dim3(kVoteThreads), 0, stream, ev, kind, rstride, ustride, R, n_units,
                           dense, kappa, status, bitmap, majority_idx);
}

hipError_t launch_consensus(const void* evidence, int kind, int64_t rstride, int64_t ustride, int R,
                            int64_t n_units, int mode, double kappa, uint8_t* status,
                            uint64_t* bitmap, int32_t* majority_idx, hipStream_t stream) {
    if (n_units <= 0) return hipSuccess;
    // Otherwise, up to 32 replicas one thread decides a unit: exact, 0.027-0.046
    // ms per 262,144 units of 64-bit fingerprints at R = 17-32 against
    // 0.044-0.046 for a wave per unit; the same results.
    // fp64 times of 17 to 32 replicas: sixteen lanes a unit, 36 us per 262,144
    // units at R = 17, 24 and 32, against 46, 38 and 43 for a thread per unit
    // (256 VGPRs); in fp32 a thread per unit is the faster one, 20-24 against
    // 30 us.  More units than sixteen lanes each can be launched for stay with a
    // thread per unit.
    if (mode == C3_STATISTICAL && kind == C3_EV_F64 && R >= stat_least(2) && R <= 32 &&
        n_units <= kGroupMaxUnits)
        return launch_stat<2>(static_cast<const char*>(evidence), kind, rstride, ustride, R, n_units,
                              kappa, status, bitmap, majority_idx, stream);
    if (R <= 32) {
        const int64_t blocks = (n_units + kVoteThreads - 1) / kVoteThreads;
        if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
        const char* e = static_cast<const char*>(evidence);
        if (R <= 4)
            launch_small<4>(e, kind, rstride, ustride, R, n_units, mode, kappa, status, bitmap,
                            majority_idx, stream, (unsigned)blocks);
        else if (R <= 8)
            launch_small<8>(e, kind, rstride, ustride, R, n_units, mode, kappa, status, bitmap,
                            majority_idx, stream, (unsigned)blocks);
        else if (R <= 16)
            launch_small<16>(e, kind, rstride, ustride, R, n_units, mode, kappa, status, bitmap,
                             majority_idx, stream, (unsigned)blocks);
        else
            launch_small<32>(e, kind, rstride, ustride, R, n_units, mode, kappa, status, bitmap,
                             majority_idx, stream, (unsigned)blocks);
        return hipGetLastError();
    }
    if (R > C3_MAX_PEERS) return hipErrorInvalidValue;
    const char* e = static_cast<const char*>(evidence);
    if (mode == C3_STATISTICAL) {
        if (R <= 64)
            return launch_stat<4>(e, kind, rstride, ustride, R, n_units, kappa, status, bitmap,
                                  majority_idx, stream);
        if (R <= 128)
            return launch_stat<8>(e, kind, rstride, ustride, R, n_units, kappa, status, bitmap,
                                  majority_idx, stream);
        if (R <= 192)
            return launch_stat<12>(e, kind, rstride, ustride, R, n_units, kappa, status, bitmap,
                                   majority_idx, stream);
        return launch_stat<16>(e, kind, rstride, ustride, R, n_units, kappa, status, bitmap,
                               majority_idx, stream);
    }
    const int64_t blocks = (n_units + kWideUnitsPerBlock - 1) / kWideUnitsPerBlock;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const unsigned nb = (unsigned)blocks;
    if (R <= 64)
        launch_exact_wide<1>(e, kind, rstride, ustride, R, n_units, status, bitmap, majority_idx, stream, nb);
    else if (R <= 128)
        launch_exact_wide<2>(e, kind, rstride, ustride, R, n_units, status, bitmap, majority_idx, stream, nb);
    else if (R <= 192)
        launch_exact_wide<3>(e, kind, rstride, ustride, R, n_units, status, bitmap, majority_idx, stream, nb);
    else
        launch_exact_wide<4>(e, kind, rstride, ustride, R, n_units, status, bitmap, majority_idx, stream, nb);
    return hipGetLastError();
}

}  // namespace c3
