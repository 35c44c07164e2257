// Temporal confirmation of C3 results for gfx950.
//
// Input: per-iteration outlier bitmaps of G peer groups (u64 per (t, g)) for
// fingerprints (exact C3) and timings (statistical C3).  Output: one verdict
// per rank, rank = r * G + g.
//
// Three forms: groups of up to 16 replicas with W <= 64 (one thread per
// segment and group), wider groups with W <= 64 (one wave per segments and
// group, one launch), and longer windows (one thread per segment and rank).
// The first and the last write partial results per (segment, rank), stored
// [segment][group][replica], which pass 2, one thread per rank, combines in
// order.
//
// Longer windows: a segment is kSeg consecutive iterations; threads are
// ordered (segment, group, replica), so the R threads of one group are
// adjacent lanes reading the same bitmap word.  The thread counts attributed
// iterations in its segment, notes the first attributed fingerprint and any
// two consecutive attributed timings (the pair (t, t + 1) belongs to the
// segment of t), and slides a window of W iterations over the window starts
// in its segment.
#include "c3_device.h"
#include "c3_internal.h"

namespace c3 {

constexpr int64_t kSeg = 64;
#ifndef C3_CONFIRM_GROUP_SEG
#define C3_CONFIRM_GROUP_SEG 32
#endif
constexpr int kGroupSeg = C3_CONFIRM_GROUP_SEG;   // segment of the per-group kernel
constexpr int kConfThreads = 256;

struct SegVerdict {
    uint32_t flags;          // bit 2: two consecutive slow iterations
    int32_t first_div;       // first attributed fingerprint iteration, -1
    uint32_t div_count;
    uint32_t slow_count;
    uint32_t max_window;
    int32_t first_window;    // first window start over the threshold, -1
};
static_assert(sizeof(SegVerdict) == 24, "segment verdict layout");

__device__ inline uint32_t bit_of(const uint64_t* bm, int64_t t, int64_t G, int64_t g, int r) {
    return (uint32_t)((bm[t * G + g] >> r) & 1ull);
}

__global__ void __launch_bounds__(kConfThreads) confirm_segment_kernel(
    const uint64_t* __restrict__ fpb, const uint64_t* __restrict__ tmb, int R, int64_t G, int64_t T,
    int64_t Wt, int64_t n_seg, SegVerdict* __restrict__ out) {
    const int64_t n_ranks = (int64_t)R * G;
    const int64_t idx = (int64_t)blockIdx.x * kConfThreads + threadIdx.x;
    if (idx >= n_ranks * n_seg) return;
    const int64_t sgi = idx / n_ranks;
    const int64_t gr = idx - sgi * n_ranks;      // g * R + r
    const int64_t g = gr / R;
    const int r = (int)(gr - g * R);
    const int64_t t0 = sgi * kSeg;
    const int64_t t1 = min(T, t0 + kSeg);
    SegVerdict v{0u, -1, 0u, 0u, 0u, -1};
    uint32_t prev = 0;
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t dv = bit_of(fpb, t, G, g, r);
        const uint32_t sl = bit_of(tmb, t, G, g, r);
        if (dv) {
            if (v.first_div < 0) v.first_div = (int32_t)t;
            ++v.div_count;
        }
        v.slow_count += sl;
        if (sl && prev) v.flags |= 4u;
        prev = sl;
    }
    // the pair (t1 - 1, t1) belongs to this segment
    if (t1 < T && prev && bit_of(tmb, t1, G, g, r)) v.flags |= 4u;
    // windows starting in [t0, min(t1, T - Wt + 1))
    const int64_t s_end = min(t1, T - Wt + 1);
    if (Wt > 0 && t0 < s_end) {
        uint32_t c = 0;
        for (int64_t t = t0; t < t0 + Wt; ++t) c += bit_of(tmb, t, G, g, r);
        for (int64_t s = t0;; ++s) {
            if (c > v.max_window) v.max_window = c;
            if (2 * (int64_t)c > Wt && v.first_window < 0) v.first_window = (int32_t)s;
            if (s + 1 >= s_end) break;
            c += bit_of(tmb, s + Wt, G, g, r);
            c -= bit_of(tmb, s, G, g, r);
        }
    }
    out[idx] = v;
}

// Groups of up to RMAX replicas with W <= 64: one thread per (segment,
// group) reads each bitmap word once and transposes it into per-replica
// 64-bit masks over iterations (lo/div: t0 + i; hi: t0 + 64 + i), then
// evaluates every replica's counts and windows with shifts and popcounts.
// Results go to the same [segment][group][replica] slots as the general
// kernel.
template <int RMAX, int SEG>
__global__ void __launch_bounds__(kConfThreads) confirm_group_kernel(
    const uint64_t* __restrict__ fpb, const uint64_t* __restrict__ tmb, int R, int64_t G, int64_t T,
    int64_t Wt, int64_t n_seg, SegVerdict* __restrict__ out) {
    const int64_t idx = (int64_t)blockIdx.x * kConfThreads + threadIdx.x;
    if (idx >= n_seg * G) return;
    const int64_t sgi = idx / G;
    const int64_t g = idx - sgi * G;
    const int64_t t0 = sgi * SEG;
    const int64_t t1 = min(T, t0 + SEG);
    // read past the segment for its windows, and t1 for the pair (t1 - 1, t1)
    const int64_t t_hi_end = min(T, t1 + (Wt > 1 ? Wt - 1 : 1));
    uint64_t div[RMAX], lo[RMAX], hi[RMAX];
#pragma unroll
    for (int r = 0; r < RMAX; ++r) div[r] = lo[r] = hi[r] = 0;
    const uint64_t* fp = fpb + t0 * G + g;
    const uint64_t* tm = tmb + t0 * G + g;
    const int nlo = (int)(t1 - t0);
    if (nlo == SEG) {
        // full segment: fixed trip count, so the loads are issued ahead
#pragma unroll 16
        for (int i = 0; i < SEG; ++i) {
            const uint64_t fw = fp[(int64_t)i * G], tw = tm[(int64_t)i * G];
#pragma unroll
            for (int r = 0; r < RMAX; ++r) {
                div[r] |= ((fw >> r) & 1ull) << i;
                lo[r] |= ((tw >> r) & 1ull) << i;
            }
        }
    } else {
        for (int i = 0; i < nlo; ++i) {
            const uint64_t fw = fp[(int64_t)i * G], tw = tm[(int64_t)i * G];
#pragma unroll
            for (int r = 0; r < RMAX; ++r) {
                div[r] |= ((fw >> r) & 1ull) << i;
                lo[r] |= ((tw >> r) & 1ull) << i;
            }
        }
    }
    const int nhi = t_hi_end > t0 + SEG ? (int)(t_hi_end - t0 - SEG) : 0;
#pragma unroll 8
    for (int i = 0; i < nhi; ++i) {
        const uint64_t tw = tm[(int64_t)(SEG + i) * G];
#pragma unroll
        for (int r = 0; r < RMAX; ++r) hi[r] |= ((tw >> r) & 1ull) << i;
    }
    const int64_t s_end = min(t1, T - Wt + 1);
    const uint64_t wmask = Wt == 64 ? ~0ull : ((1ull << Wt) - 1);
    const uint64_t seg_mask = SEG == 64 ? ~0ull : ((1ull << SEG) - 1);
    SegVerdict* o = out + sgi * (int64_t)R * G + g * R;
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (r >= R) break;
        // 128-bit run of timing bits: bit i is iteration t0 + i
        const uint64_t b0 = SEG == 64 ? lo[r] : (lo[r] | (hi[r] << (SEG & 63)));
        const uint64_t b1 = SEG == 64 ? hi[r] : (hi[r] >> ((64 - SEG) & 63));
        SegVerdict v{0u, -1, 0u, 0u, 0u, -1};
        v.div_count = (uint32_t)__builtin_popcountll(div[r]);
        v.first_div = div[r] ? (int32_t)(t0 + __builtin_ctzll(div[r])) : -1;
        v.slow_count = (uint32_t)__builtin_popcountll(lo[r]);
        // pairs (t, t + 1) with t in the segment; bits past T are zero
        const uint64_t pairs = b0 & ((b0 >> 1) | (b1 << 63)) & seg_mask;
        if (pairs != 0) v.flags |= 4u;
        for (int64_t s0 = t0; s0 < s_end; ++s0) {
            const int off = (int)(s0 - t0);
            const uint64_t w = off == 0 ? b0 : ((b0 >> off) | (b1 << (64 - off)));
            const uint32_t c = (uint32_t)__builtin_popcountll(w & wmask);
            if (c > v.max_window) v.max_window = c;
            if (2 * (int64_t)c > Wt && v.first_window < 0) v.first_window = (int32_t)s0;
        }
        o[r] = v;
    }
}

__global__ void __launch_bounds__(kConfThreads) confirm_combine_kernel(
    const SegVerdict* __restrict__ seg, int R, int64_t G, int64_t n_ranks, int64_t n_seg,
    c3_rank_verdict_t* __restrict__ verdicts) {
    const int64_t rank = (int64_t)blockIdx.x * kConfThreads + threadIdx.x;
    if (rank >= n_ranks) return;
    const int64_t r = rank / G;
    const int64_t g = rank - r * G;
    const int64_t gr = g * R + r;               // position inside a segment's block
    uint32_t fl = 0, dc = 0, sc = 0, mw = 0;
    int32_t fd = -1, fw = -1;
#pragma unroll 4
    for (int64_t s = 0; s < n_seg; ++s) {
        const SegVerdict v = seg[s * n_ranks + gr];
        fl |= v.flags;
        dc += v.div_count;
        sc += v.slow_count;
        mw = max(mw, v.max_window);
        if (fd < 0) fd = v.first_div;
        if (fw < 0) fw = v.first_window;
    }
    if (fw >= 0) fl |= C3_RANK_STRAGGLER;
    if (fd >= 0) fl |= C3_RANK_PROTOCOL;
    c3_rank_verdict_t out;
    out.flags = fl;
    out.first_divergent_iter = fd;
    out.divergent_count = dc;
    out.slow_count = sc;
    out.max_window_slow = mw;
    out.first_straggler_window = fw;
    verdicts[rank] = out;
}

// Groups of 17 to 64 replicas with W <= 64, in one launch.  A wave takes a
// group's segments of 64 iterations: lane i loads the words of iteration t0 +
// i, and lane r collects replica r's bits over the iterations into 64-bit
// masks.  The words of most groups are nearly all zero, so few of them are
// walked, broadcast by readlane; those of a group with a slow or diverged rank
// are set at every iteration, and such a group's walk was the kernel's time
// (128 groups of 32 over 512 iterations, one with a slow and a diverged rank:
// 9.8 us), so they are transposed in six levels of lane exchanges (4.8 us;
// without outliers 3.5).  A window's count rises only where a set bit enters, so the largest
// count and the first window over the threshold are those of windows ending
// at a set bit or starting the segment: a lane evaluates those, and only
// where they could change what it already has.  `sw` waves share a group's
// segments, strided, and meet in LDS; the workgroup's other waves take
// adjacent groups, whose words share cache lines, and workgroups are dealt so
// that neighbours run on one XCD.  The thread per (segment, rank) of before
// walked 191 words and 64 windows each: 38.8 us, and 5.9 us to combine, for
// 128 groups of 32 over 512 iterations.
constexpr int kWaveConfWaves = 8;

// Most non-zero words of 64 that are walked one by one: about what a transpose
// costs.
constexpr int kGatherWords = 6;

// The 64 x 64 bit matrix whose row i lane i holds, transposed: blocks of 32,
// 16, ... 1 change places between the lanes that differ in that bit.
template <int S>
__device__ __forceinline__ uint32_t transpose_level(uint32_t x, uint32_t mask, int lane) {
    const uint32_t p = row_xor_u32<S>(x);
    const uint32_t keep = (lane & S) != 0 ? ~mask : mask;
    const uint32_t t = (lane & S) != 0 ? p >> S : p << S;
    return (x & keep) | (t & ~keep);
}
__device__ __forceinline__ uint64_t transpose64(uint64_t w, int lane) {
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)w, (uint32_t)(w >> 32), false, false);
    uint32_t x[2] = {h[0], h[1]};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // [0], [1]: the word of the even and of the odd row of the pair
        const auto q = __builtin_amdgcn_permlane16_swap(x[i], x[i], false, false);
        x[i] = (lane & 16) == 0 ? (q[0] & 0xFFFFu) | (q[1] << 16) : (q[0] >> 16) | (q[1] & 0xFFFF0000u);
        x[i] = transpose_level<8>(x[i], 0x00FF00FFu, lane);
        x[i] = transpose_level<4>(x[i], 0x0F0F0F0Fu, lane);
        x[i] = transpose_level<2>(x[i], 0x33333333u, lane);
        x[i] = transpose_level<1>(x[i], 0x55555555u, lane);
    }
    return ((uint64_t)x[1] << 32) | x[0];
}

struct RankAcc {
    uint32_t flags, dc, sc, mw;
    int32_t fd, fw;
};

__global__ void __launch_bounds__(64 * kWaveConfWaves) confirm_wave_kernel(
    const uint64_t* __restrict__ fpb, const uint64_t* __restrict__ tmb, int R, int64_t G, int64_t T,
    int Wt, int sw, c3_rank_verdict_t* __restrict__ verdicts) {
    __shared__ RankAcc acc[kWaveConfWaves][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int gw = kWaveConfWaves / sw;                 // groups per workgroup
    const unsigned nb = gridDim.x;
    const unsigned blk = nb % 8u != 0u ? blockIdx.x
                                       : (blockIdx.x % 8u) * (nb / 8u) + blockIdx.x / 8u;
    const int64_t g = (int64_t)blk * gw + wave / sw;
    const int part = wave % sw;
    RankAcc a{0u, 0u, 0u, 0u, -1, -1};
    if (g < G) {
        const int64_t n_seg = (T + 63) / 64;
        // Iteration t's word, 0 past the end.  A lane's bits past T stay 0.
        auto word = [&](const uint64_t* bm, int64_t t) { return t < T ? bm[t * G + g] : 0ull; };
        // lane r's bits over the 64 words the lanes hold: a walk of the
        // non-zero words, a few in a sound group, or a transpose
        auto gather = [&](uint64_t w) {
            uint64_t m = 0, set = ballot64(w != 0ull);
            if (__builtin_popcountll(set) > kGatherWords) return transpose64(w, lane);
            for (; set != 0ull; set &= set - 1ull) {
                const int i = __builtin_ctzll(set);
                m |= ((readlane_u64(w, i) >> lane) & 1ull) << i;
            }
            return m;
        };
        const uint64_t wmask = Wt == 64 ? ~0ull : ((1ull << Wt) - 1ull);
        // words of the segment, and of the iterations its last windows and
        // its last pair (t1 - 1, t1) reach into
        const int past = Wt > 1 ? Wt - 1 : 1;
        uint64_t fw0 = word(fpb, (int64_t)part * 64 + lane);
        uint64_t tw0 = word(tmb, (int64_t)part * 64 + lane);
        uint64_t tw1 = lane < past ? word(tmb, (int64_t)part * 64 + 64 + lane) : 0ull;
        for (int64_t sg = part; sg < n_seg; sg += sw) {
            const uint64_t f = fw0, t_in = tw0, t_past = tw1;
            const int64_t nx = (sg + sw) * 64 + lane;   // the next segment's words, under this one
            if (sg + sw < n_seg) {
                fw0 = word(fpb, nx);
                tw0 = word(tmb, nx);
                tw1 = lane < past ? word(tmb, nx + 64) : 0ull;
            }
            const int64_t t0 = sg * 64;
            const uint64_t div = gather(f), lo = gather(t_in), hi = gather(t_past);
            if (div != 0ull && a.fd < 0) a.fd = (int32_t)(t0 + __builtin_ctzll(div));
            a.dc += (uint32_t)__builtin_popcountll(div);
            const uint32_t in = (uint32_t)__builtin_popcountll(lo);
            a.sc += in;
            if ((lo & (lo >> 1)) != 0ull || ((lo >> 63) & hi & 1ull) != 0ull) a.flags |= C3_RANK_CONSEC2;
            // windows starting at t0 + off, off < n_off, inside the T iterations
            const int64_t t1 = t0 + 64 < T ? t0 + 64 : T;
            const int64_t s_end = t1 < T - Wt + 1 ? t1 : T - Wt + 1;
            const int n_off = s_end > t0 ? (int)(s_end - t0) : 0;
            const uint32_t all = in + (uint32_t)__builtin_popcountll(hi);
            const uint32_t cap = all < (uint32_t)Wt ? all : (uint32_t)Wt;
            if (n_off > 0 && (cap > a.mw || (2u * cap > (uint32_t)Wt && a.fw < 0))) {
                auto window = [&](int off) {
                    const uint64_t w = off == 0 ? lo : ((lo >> off) | (hi << (64 - off)));
                    const uint32_t c = (uint32_t)__builtin_popcountll(w & wmask);
                    a.mw = c > a.mw ? c : a.mw;
                    if (2u * c > (uint32_t)Wt && a.fw < 0) a.fw = (int32_t)(t0 + off);
                };
                window(0);
                // windows ending at a set bit p = Wt .. Wt + n_off - 2
                for (int half = 0; half < 2; ++half) {
                    uint64_t ev = half == 0 ? lo : hi;
                    const int base = 64 * half;
                    const int from = Wt - base, to = Wt + n_off - 1 - base;     // [from, to)
                    if (from >= 64 || to <= 0) continue;
                    if (from > 0) ev &= ~0ull << from;
                    if (to < 64) ev &= (1ull << to) - 1ull;
                    // a full window: no later one raises the maximum or comes first
                    while (ev != 0ull && !(a.mw >= (uint32_t)Wt && a.fw >= 0)) {
                        const int p = base + __builtin_ctzll(ev);
                        ev &= ev - 1ull;
                        window(p - Wt + 1);
                    }
                }
            }
        }
    }
    acc[wave][lane] = a;
    __syncthreads();
    if (part != 0 || g >= G || lane >= R) return;
    for (int k = 1; k < sw; ++k) {
        const RankAcc b = acc[wave + k][lane];
        a.flags |= b.flags;
        a.dc += b.dc;
        a.sc += b.sc;
        a.mw = max(a.mw, b.mw);
        a.fd = (a.fd < 0 || (b.fd >= 0 && b.fd < a.fd)) ? b.fd : a.fd;
        a.fw = (a.fw < 0 || (b.fw >= 0 && b.fw < a.fw)) ? b.fw : a.fw;
    }
    if (a.fw >= 0) a.flags |= C3_RANK_STRAGGLER;
    if (a.fd >= 0) a.flags |= C3_RANK_PROTOCOL;
    c3_rank_verdict_t v;
    v.flags = a.flags;
    v.first_divergent_iter = a.fd;
    v.divergent_count = a.dc;
    v.slow_count = a.sc;
    v.max_window_slow = a.mw;
    v.first_straggler_window = a.fw;
    verdicts[(int64_t)lane * G + g] = v;
}

size_t confirm_ws_bytes(int R, int64_t G, int64_t T) {
    const int64_t seg_len = kGroupSeg < kSeg ? kGroupSeg : kSeg;
    const int64_t n_seg = T > 0 ? (T + seg_len - 1) / seg_len : 1;
    return (size_t)(n_seg * (int64_t)R * G * (int64_t)sizeof(SegVerdict)) + 256;
}

hipError_t launch_confirm(const uint64_t* fp_bitmap, const uint64_t* time_bitmap, int R, int64_t G,
                          int64_t T, int window, c3_rank_verdict_t* verdicts, void* ws,
                          hipStream_t stream) {
    const int64_t n_ranks = (int64_t)R * G;
    if (n_ranks == 0) return hipSuccess;
    const int64_t Wt = (int64_t)window < T ? (int64_t)window : T;
    const int64_t wave_segs = (T + 63) / 64;
    const int sw = wave_segs >= 8 ? 8 : wave_segs >= 4 ? 4 : wave_segs >= 2 ? 2 : 1;
    const int64_t gw = kWaveConfWaves / sw;
    const int64_t blocks = (G + gw - 1) / gw;
    // (more groups than a grid of fewer than 2^32 threads has waves for: two launches)
    if (R > 16 && Wt <= 64 && T > 0 && blocks * 64 * kWaveConfWaves < ((int64_t)1 << 32)) {
        hipLaunchKernelGGL(confirm_wave_kernel, dim3((unsigned)blocks), dim3(64 * kWaveConfWaves), 0,
                           stream, fp_bitmap, time_bitmap, R, G, T, (int)Wt, sw, verdicts);
        return hipGetLastError();
    }
    SegVerdict* seg = static_cast<SegVerdict*>(ws);
    const bool by_group = R <= 16 && Wt <= 64;
    const int64_t seg_len = by_group ? kGroupSeg : kSeg;
    const int64_t n_seg = T > 0 ? (T + seg_len - 1) / seg_len : 1;
    const int64_t threads1 = (by_group ? G : n_ranks) * n_seg;
    const int64_t blocks1 = (threads1 + kConfThreads - 1) / kConfThreads;
    if (blocks1 > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (by_group && R <= 8)
        hipLaunchKernelGGL((confirm_group_kernel<8, kGroupSeg>), dim3((unsigned)blocks1),
                           dim3(kConfThreads), 0, stream, fp_bitmap, time_bitmap, R, G, T, Wt, n_seg,
                           seg);
    else if (by_group)
        hipLaunchKernelGGL((confirm_group_kernel<16, kGroupSeg>), dim3((unsigned)blocks1),
                           dim3(kConfThreads), 0, stream, fp_bitmap, time_bitmap, R, G, T, Wt, n_seg,
                           seg);
    else
        hipLaunchKernelGGL(confirm_segment_kernel, dim3((unsigned)blocks1), dim3(kConfThreads), 0,
                           stream, fp_bitmap, time_bitmap, R, G, T, Wt, n_seg, seg);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t blocks2 = (n_ranks + kConfThreads - 1) / kConfThreads;
    hipLaunchKernelGGL(confirm_combine_kernel, dim3((unsigned)blocks2), dim3(kConfThreads), 0, stream,
                       seg, R, G, n_ranks, n_seg, verdicts);
    return hipGetLastError();
}

}  // namespace c3
