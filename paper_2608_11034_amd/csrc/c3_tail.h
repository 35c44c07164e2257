// Votes and lists of a small record table in one workgroup: the last step of
// c3_check on small plans and of the optimizer-boundary check.
#pragma once

#include "c3_device.h"
#include "c3_internal.h"
#include "c3_vote_row.h"

namespace c3 {

constexpr int kTailThreads = 1024;
constexpr int kTailMaxChunks = 256;
constexpr int kTailMaxRecords = 1024;

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ inline uint64_t wave_inclusive_scan(uint64_t x, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t y = shfl_u64(x, lane >= d ? lane - d : lane);
        if (lane >= d) x += y;
    }
    return x;
}

__device__ inline void outlier_from(c3_outlier_t& o, int64_t u, int r, int mj,
                                    const c3_chunk_record_t& a, const c3_chunk_record_t& b) {
    o.chunk = u;
    o.replica = r;
    o.majority_replica = mj;
    o.nan_count[0] = a.nan_count;
    o.nan_count[1] = b.nan_count;
    o.inf_count[0] = a.inf_count;
    o.inf_count[1] = b.inf_count;
    o.absmax[0] = a.absmax;
    o.absmax[1] = b.absmax;
    o.sum[0] = a.sum;
    o.sum[1] = b.sum;
    o.sumsq[0] = a.sumsq;
    o.sumsq[1] = b.sumsq;
}

// exact_vote_row's rule with the signatures read where they are (R > 32: 64 of
// them would take 128 registers of a 1,024-thread workgroup's 128).
template <typename Sig>
__device__ inline UnitVote exact_vote_by(const Sig& sig, int R) {
    const uint64_t e0 = sig(0);
    uint64_t maj = 0;
    for (int r = 0; r < R; ++r) maj |= (uint64_t)(sig(r) == e0) << r;
    if (2 * __builtin_popcountll(maj) <= R) {
        uint64_t cand = e0;
        int cnt = 0;
        for (int r = 0; r < R; ++r) {
            const uint64_t e = sig(r);
            if (cnt == 0) cand = e;
            cnt += e == cand ? 1 : -1;
        }
        maj = 0;
        for (int r = 0; r < R; ++r) maj |= (uint64_t)(sig(r) == cand) << r;
    }
    if (2 * __builtin_popcountll(maj) <= R) return UnitVote{0ull, -1, (uint8_t)C3_INCONCLUSIVE};
    const uint64_t valid = R == 64 ? ~0ull : ((1ull << R) - 1);
    const uint64_t b = valid & ~maj;
    return UnitVote{b, (int32_t)__builtin_ctzll(maj), b ? (uint8_t)C3_ATTRIBUTED : (uint8_t)C3_AGREE};
}

// rec[r * C + u] (in LDS, being written by the workgroup): one thread per
// chunk votes with exact_vote_row, the rule c3_consensus applies, on the
// signatures; a scan over the chunks of their outlier and undecided counts
// gives each chunk's thread the place of its entries (chunk ascending,
// replica ascending within a chunk, both replicas' summaries), and thread 0
// writes the counts.  C <= kTailMaxChunks, R <= 64, R * C <= kTailMaxRecords.
__device__ inline void tail_votes_and_lists(const c3_chunk_record_t* rec, int R, int C,
                                            const TailOut& out) {
    __shared__ uint64_t wave_total[kTailMaxChunks / 64];
    __syncthreads();
    const int u = threadIdx.x;              // threads past C only meet the barrier
    UnitVote v{0ull, -1, (uint8_t)C3_AGREE};
    if (u < C) {
        if (R <= 16) {
            uint64_t e[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) e[r] = r < R ? rec[r * C + u].sig : 0ull;
            v = exact_vote_row<16>(e, R);
        } else if (R <= 32) {
            uint64_t e[32];
#pragma unroll
            for (int r = 0; r < 32; ++r) e[r] = r < R ? rec[r * C + u].sig : 0ull;
            v = exact_vote_row<32>(e, R);
        } else {
            v = exact_vote_by([&](int r) { return rec[r * C + u].sig; }, R);
        }
        out.status[u] = v.status;
        out.bitmap[u] = v.bitmap;
        out.majority[u] = v.majority;
    }
    // counts packed as outliers (24 bits: at most 256 chunks x 63), undecided
    // and attributed chunks (20 bits each)
    const bool und = u < C && v.status == C3_INCONCLUSIVE;
    const uint64_t n_o = u < C && !und ? (uint64_t)__builtin_popcountll(v.bitmap) : 0ull;
    const uint64_t packed = n_o | ((uint64_t)und << 24) | ((uint64_t)(n_o != 0ull) << 44);
    const int lane = u & 63, wave = u >> 6;
    const uint64_t incl = wave_inclusive_scan(packed, lane);
    if (lane == 63 && wave < kTailMaxChunks / 64) wave_total[wave] = incl;
    __syncthreads();
    uint64_t before = 0ull, total = 0ull;
#pragma unroll
    for (int w = 0; w < kTailMaxChunks / 64; ++w) {
        const uint64_t t = wave_total[w];
        before += w < wave ? t : 0ull;
        total += t;
    }
    const uint64_t excl = before + incl - packed;
    int64_t po = (int64_t)(excl & 0xFFFFFFull);
    const int64_t pu = (int64_t)((excl >> 24) & 0xFFFFFull);
    for (uint64_t b = n_o ? v.bitmap : 0ull; b != 0ull && po < out.out_cap; b &= b - 1ull, ++po) {
        const int r = __builtin_ctzll(b);
        c3_outlier_t o;
        outlier_from(o, u, r, v.majority, rec[r * C + u], rec[v.majority * C + u]);
        out.outliers[po] = o;
    }
    if (und && pu < out.und_cap) out.undecided[pu] = u;
    if (u == 0) {
        out.counts[0] = (int64_t)(total & 0xFFFFFFull);
        out.counts[1] = (int64_t)((total >> 24) & 0xFFFFFull);
        out.counts[2] = (int64_t)((total >> 44) & 0xFFFFFull);
    }
}

}  // namespace c3
