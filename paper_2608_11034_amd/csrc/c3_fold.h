// Folding bytes into C3SIG-1 accumulators and numerical summaries: one lane's
// share of a tile, the wave reduction, the combination of quarters and tiles,
// and the chunk record.  Shared by the streaming signature kernels
// (c3_signature.hip) and the optimizer-boundary kernel (c3_optimizer.hip).
#pragma once

#include "c3_device.h"
#include "c3_internal.h"

namespace c3 {

constexpr int kRedoLoads = 8;   // loads in flight where a lane classifies its elements

struct LaneKeys {
    uint32_t k0, k1, k2, k3, k4, k5;
};

__device__ inline LaneKeys lane_keys(int lane) {
    LaneKeys K;
    K.k0 = nh_key(4u * lane + 0u);
    K.k1 = nh_key(4u * lane + 1u);
    K.k2 = nh_key(4u * lane + 2u);
    K.k3 = nh_key(4u * lane + 3u);
    K.k4 = nh_key(4u * lane + 4u);
    K.k5 = nh_key(4u * lane + 5u);
    return K;
}

// beta of block b (wave-uniform, so it stays in a scalar register)
__device__ inline uint32_t block_beta(uint32_t b) { return b * kBlockMul; }

// m + k + beta as one three-input add with beta as the scalar operand.  The
// compiler would otherwise re-associate to m + (k + beta) and spend a
// separate add on each of the six key sums per block.
__device__ inline uint32_t add3(uint32_t m, uint32_t k, uint32_t beta) {
    uint32_t r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(k), "s"(beta));
    return r;
}

// NH over one 16-byte segment (two word pairs) at key offset 4 * lane.
__device__ inline void nh16(const u32x4 v, const LaneKeys& K, uint32_t beta, uint64_t& A,
                            uint64_t& B) {
    A += (uint64_t)add3(v.x, K.k0, beta) * (uint64_t)add3(v.y, K.k1, beta);
    B += (uint64_t)add3(v.x, K.k2, beta) * (uint64_t)add3(v.y, K.k3, beta);
    A += (uint64_t)add3(v.z, K.k2, beta) * (uint64_t)add3(v.w, K.k3, beta);
    B += (uint64_t)add3(v.z, K.k4, beta) * (uint64_t)add3(v.w, K.k5, beta);
}

__device__ inline double f16_to_f64(uint32_t h) {
    _Float16 x = __builtin_bit_cast(_Float16, (uint16_t)h);
    return (double)(float)x;
}

// ---------------------------------------------------------------------------
// fast statistics: no classification.  `mf` collects the largest magnitude as
// an fp32 value (every fp32, bf16 and fp16 value is one exactly); a NaN or
// Inf may poison it, but such a lane takes the classifying path below, which
// starts over.
// ---------------------------------------------------------------------------
// max(|a|, |b|, |c|) in one instruction (abs source modifiers); NaN
// propagates, which only matters on lanes the classifying path redoes.
__device__ inline float absmax3(float a, float b, float c) {
    float r;
    asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// fp64 sums of a lane's elements in one quarter of a tile.
//
// The squares of bf16 and fp16 elements have at most 22 bits and no chain of a
// tile rounds them.  Those of fp32 elements have 48, their lowest bits are
// alike (an odd number's square is 1 mod 8), and a plain chain rounds most of
// them down: 2-norm of the relative error of a chunk of N(0, 1) elements 2.5e-16
// over 64 elements a lane (64 KiB tiles), 8.8e-16 over 256 (256 KiB).
//
// Chunks that are powers of two, and tiles that a caller asks for, have tiles
// that are powers of two and plain chains.  Other chunks have larger tiles than
// the power of two that divides them (100 KiB in place of 4), and folds make up
// for it (FOLD, folded_tiles): the even and the odd elements have a chain each,
// and after every kFoldBlocks blocks of the quarter, 8 elements a chain, their
// sum goes into a compensated pair.  Error of chunks of 48, 100, 160, 500 and
// 1000 KiB in tiles of the power of two 8.3e-17, 6.2e-17, 9.3e-17, 5.2e-17 and
// 6.4e-17, in the larger tiles 1.6e-16, 2.9e-16, 5.4e-16, 8.6e-16 and 8.8e-16,
// with folds 7.7e-17, 6.5e-17, 8.1e-17, 5.2e-17 and 5.9e-17 (folds after 16
// blocks 2e-16; rounding the exact sum once 4e-17 to 6e-17).  That is 7 more fp64
// instructions to 32, within the noise of a call: 3 GB in 1000 KiB chunks 448 /
// 445 us, 805 MB in 96 KiB chunks 125.0 / 124.8, 403 MB in 33 KiB chunks, a wave
// each, 82.9 / 84.0.  The sums themselves add 24-bit values and round next to
// nothing.
constexpr int kFoldBlocks = 4;

template <int DT, bool FOLD>
struct LaneSums {
    double s = 0.0, q = 0.0;
    __device__ __forceinline__ void add(double d, int) {
        s += d;
        q = __fma_rn(d, d, q);
    }
    __device__ __forceinline__ void fold() {}
    __device__ __forceinline__ double squares() { return q; }
};
template <>
struct LaneSums<C3_F32, true> {
    double s = 0.0, q[2] = {0.0, 0.0}, hi = 0.0, lo = 0.0;
    __device__ __forceinline__ void add(double d, int i) {
        s += d;
        q[i & 1] = __fma_rn(d, d, q[i & 1]);
    }
    __device__ __forceinline__ void fold() {
        double t, e;
        two_sum(hi, q[0] + q[1], t, e);
        hi = t;
        lo += e;
        q[0] = q[1] = 0.0;
    }
    // (with nothing in the chains the last fold changes nothing)
    __device__ __forceinline__ double squares() {
        fold();
        return hi + lo;
    }
};

template <int DT, bool FOLD>
__device__ inline void stats_fast(const u32x4 v, LaneSums<DT, FOLD>& a, float& mf) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    if constexpr (DT == C3_F32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a.add((double)__uint_as_float(w[i]), i);
        mf = absmax3(mf, absmax3(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2])),
                     __uint_as_float(w[3]));
    } else if constexpr (DT == C3_BF16 || DT == C3_F16) {
        float x[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (DT == C3_BF16) {
                x[2 * i] = __uint_as_float(w[i] << 16);
                x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
            } else {
                x[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] & 0xFFFFu));
                x[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] >> 16));
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) a.add((double)x[i], i);
        mf = absmax3(absmax3(x[0], x[1], x[2]), absmax3(x[3], x[4], x[5]), absmax3(x[6], x[7], mf));
    }
}

// magnitude bits of the type from the fp32 value of a finite magnitude
template <int DT>
__device__ inline uint32_t magnitude_bits(float mf) {
    if constexpr (DT == C3_BF16) return __float_as_uint(mf) >> 16;  // exact: a bf16 value
    if constexpr (DT == C3_F16) return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)mf);
    return __float_as_uint(mf);
}

// slow statistics: classify each element; `mx` is a plain magnitude.  A
// non-finite element counts as +0, which changes no sum (they start at +0,
// so none is ever -0), and there are no branches: one lane redoes its column
// of the tile while the wave waits.
template <int DT, bool FOLD>
__device__ inline void stats_slow(const u32x4 v, LaneSums<DT, FOLD>& a, uint32_t& mx, uint32_t& nan_c,
                                  uint32_t& inf_c) {
    constexpr uint32_t inf_bits = DT == C3_F32 ? 0x7F800000u : DT == C3_BF16 ? 0x7F80u : 0x7C00u;
    constexpr int N = DT == C3_F32 ? 4 : 8;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t x = w[DT == C3_F32 ? i : i >> 1];
        if constexpr (DT != C3_F32) x = (i & 1) ? x >> 16 : x & 0xFFFFu;
        const uint32_t mag = x & (DT == C3_F32 ? 0x7FFFFFFFu : 0x7FFFu);
        const bool fin = mag < inf_bits;
        nan_c += mag > inf_bits;
        inf_c += mag == inf_bits;
        x = fin ? x : 0u;
        mx = max(mx, fin ? mag : 0u);
        const double d = DT == C3_F32 ? (double)__uint_as_float(x)
                         : DT == C3_BF16 ? (double)__uint_as_float(x << 16) : f16_to_f64(x);
        a.add(d, i);
    }
}

// Tail segment of a tile: bytes [0, rem) of a 16-byte segment, rest zero.
__device__ inline u32x4 load_partial(const uint8_t* p, uint32_t rem) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    for (uint32_t b = 0; b < rem; ++b) w[b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
    u32x4 v;
    v.x = w[0];
    v.y = w[1];
    v.z = w[2];
    v.w = w[3];
    return v;
}

// A lane's share of a tile.  The sums are kept in quarters: quarter q holds
// blocks q, q + 4, ... of the tile, in ascending order and folded after the
// same ones, whether one wave folds all four (NQ = 4) or four waves one each
// (NQ = 1), so the sums have the same bits either way.
template <int NQ>
struct LaneFold {
    uint64_t A, B;
    double s[NQ], q[NQ];
    uint32_t mx, nan_c, inf_c;
};

// Fold of `len` bytes of a tile by NW waves (4, or 1: the whole tile by one):
// blocks wave, wave + NW, ...
// Full blocks are read with raw buffer loads: the resource is the tile (a
// wave-uniform base, `len` bytes), the scalar offset the block, the vector
// offset the lane's 16 bytes, so no load spends vector instructions on its
// address.  Each block's beta is pinned in a scalar register, so every key
// sum is one three-input add.
template <int DT, int U, int NW, bool FOLD>
__device__ inline LaneFold<4 / NW> fold_lane(const uint8_t* tile, uint32_t len, uint32_t blk0,
                                             const LaneKeys& K, int wave, int lane) {
    constexpr int NQ = 4 / NW;
    static_assert((NW == 1 || NW == 4) && U % (NQ * kFoldBlocks) == 0 && kRedoLoads % kFoldBlocks == 0,
                  "quarters of a tile");
    LaneFold<NQ> f;
    f.A = f.B = 0;
    f.mx = f.nan_c = f.inf_c = 0u;
    LaneSums<DT, FOLD> a[NQ];
    float mf = 0.0f;
    const uint32_t off = (uint32_t)lane * 16u;
    const int nfull = (int)(len >> 10);
    const uint32_t tail = len & 1023u;
    const __amdgpu_buffer_rsrc_t rs = tile_resource(tile, len);
    int k = wave;
    // k - wave is a multiple of NW U in both loops, so load u of a batch
    // belongs to quarter u % NQ, as its block u / NQ of the batch
    auto take = [&](const u32x4 v, int u) {
        stats_fast<DT>(v, a[u % NQ], mf);
        // blocks and folds one after another: side by side their chains take
        // 128 registers and scratch where 97 do
        if constexpr (DT == C3_F32 && FOLD && NW == 4) __builtin_amdgcn_sched_barrier(0);
        if (u / NQ % kFoldBlocks == kFoldBlocks - 1) {
            a[u % NQ].fold();
            if constexpr (DT == C3_F32 && FOLD && NW == 4) __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (; k + NW * (U - 1) < nfull; k += NW * U) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load16_buf(rs, off, (uint32_t)(k + NW * u) << 10);
        // keep all U loads in flight before the first use
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t beta = block_beta(blk0 + (uint32_t)(k + NW * u));
            nh16(v[u], K, beta, f.A, f.B);
            take(v[u], u);
        }
    }
    if (k < nfull) {
        // fewer than U blocks left for this wave: one more batch, all loads in
        // flight together; the tests are wave-uniform (scalar branches).
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + NW * u < nfull) v[u] = load16_buf(rs, off, (uint32_t)(k + NW * u) << 10);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + NW * u < nfull) {
                nh16(v[u], K, block_beta(blk0 + (uint32_t)(k + NW * u)), f.A, f.B);
                take(v[u], u);
            }
        }
    }
    const bool has_tail = tail != 0u && nfull % NW == wave && off < tail;
    if (has_tail) {
        const uint8_t* seg = tile + ((size_t)nfull << 10) + off;
        u32x4 v = (off + 16u <= tail) ? load16(reinterpret_cast<const u32x4*>(seg))
                                      : load_partial(seg, tail - off);
        nh16(v, K, (blk0 + (uint32_t)nfull) * kBlockMul, f.A, f.B);
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            if (nfull % NQ == i) stats_fast<DT>(v, a[i], mf);
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        f.s[i] = a[i].s;
        f.q[i] = a[i].squares();
    }
    if constexpr (DT != C3_RAW) {
        bool finite = true;
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            finite = finite && __builtin_isfinite(f.s[i]) && __builtin_isfinite(f.q[i]);
        if (!finite) {
            // rare: this lane saw a NaN or Inf; redo its statistics classifying
            f.mx = 0u;
            for (int i = 0; i < NQ; ++i) {
                LaneSums<DT, FOLD> ai;
                for (int kk = wave + i; kk < nfull; kk += 4 * kRedoLoads) {
                    u32x4 v[kRedoLoads];
#pragma unroll
                    for (int u = 0; u < kRedoLoads; ++u)
                        if (kk + 4 * u < nfull)
                            v[u] = load16_buf(rs, off, (uint32_t)(kk + 4 * u) << 10);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < kRedoLoads; ++u)
                        if (kk + 4 * u < nfull) {
                            stats_slow<DT>(v[u], ai, f.mx, f.nan_c, f.inf_c);
                            if (u % kFoldBlocks == kFoldBlocks - 1) ai.fold();
                        }
                }
                if (has_tail && nfull % NQ == i) {
                    const uint8_t* seg = tile + ((size_t)nfull << 10) + off;
                    u32x4 v = (off + 16u <= tail) ? load16(reinterpret_cast<const u32x4*>(seg))
                                                  : load_partial(seg, tail - off);
                    stats_slow<DT>(v, ai, f.mx, f.nan_c, f.inf_c);
                }
                const double qi = ai.squares();
#pragma unroll
                for (int j = 0; j < NQ; ++j)
                    if (j == i) {
                        f.s[j] = ai.s;
                        f.q[j] = qi;
                    }
            }
        } else {
            f.mx = magnitude_bits<DT>(mf);
        }
    }
    return f;
}

// Lanes meet in a fixed six-level butterfly (lane distances 32 to 1) of plain
// fp64 adds (error at most 6 ulp of the sum of magnitudes); quarters and tiles
// meet with compensation.
__device__ inline void reduce_counts(TilePartial& p, uint32_t mx, uint32_t nan_c, uint32_t inf_c) {
    p.pad = 0u;
    p.maxbits = wave_max_u32(mx);
    p.nan_count = nan_c;
    p.inf_count = inf_c;
    if (ballot64(nan_c != 0u || inf_c != 0u) != 0ull) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            p.nan_count += shfl_xor_u32(p.nan_count, m);
            p.inf_count += shfl_xor_u32(p.inf_count, m);
        }
    }
}

// One quarter of a tile (a wave of four): its partial, in every lane.
__device__ inline TilePartial wave_reduce(const LaneFold<1>& f) {
    TilePartial p;
    // A and B, sum and sum of squares side by side: lanes 0-31 end with the
    // first, lanes 32-63 with the second
    uint64_t ab = fold32(f.A, f.B);
    double sq = fold32(f.s[0], f.q[0]);
    ab = row_sum(fold16(ab, ab));
    sq = row_sum(fold16(sq, sq));
    p.A = readlane_u64(ab, 0);
    p.B = readlane_u64(ab, 32);
    from_bits(readlane_u64(bits_of(sq), 0), p.s);
    from_bits(readlane_u64(bits_of(sq), 32), p.q);
    p.sc = p.qc = 0.0;
    reduce_counts(p, f.mx, f.nan_c, f.inf_c);
    return p;
}

__device__ inline void partial_add(TilePartial& a, const TilePartial& b) {
    a.A += b.A;
    a.B += b.B;
    comp_add(a.s, a.sc, b.s, b.sc);
    comp_add(a.q, a.qc, b.q, b.qc);
    a.maxbits = max(a.maxbits, b.maxbits);
    a.nan_count += b.nan_count;
    a.inf_count += b.inf_count;
}

// A whole tile (one wave): the four quarters' sums meet as those of four
// waves do.
__device__ inline TilePartial wave_reduce(const LaneFold<4>& f) {
    TilePartial p;
    uint64_t ab = fold32(f.A, f.B);
    ab = row_sum(fold16(ab, ab));
    p.A = readlane_u64(ab, 0);
    p.B = readlane_u64(ab, 32);
    // row i of 16 lanes ends with quarter i
    const double s = row_sum(fold16(fold32(f.s[0], f.s[2]), fold32(f.s[1], f.s[3])));
    const double q = row_sum(fold16(fold32(f.q[0], f.q[2]), fold32(f.q[1], f.q[3])));
    from_bits(readlane_u64(bits_of(s), 0), p.s);
    from_bits(readlane_u64(bits_of(q), 0), p.q);
    p.sc = p.qc = 0.0;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        double si, qi;
        from_bits(readlane_u64(bits_of(s), 16 * i), si);
        from_bits(readlane_u64(bits_of(q), 16 * i), qi);
        comp_add(p.s, p.sc, si, 0.0);
        comp_add(p.q, p.qc, qi, 0.0);
    }
    reduce_counts(p, f.mx, f.nan_c, f.inf_c);
    return p;
}

// Combination of a chunk's tile partials, a fixed tree: partial x belongs to
// lane x mod 16 of a group of sixteen, each lane adds its own in ascending
// order, and the lanes meet at distances 8, 4, 2 and 1.  partial_merge gives
// the same bits for (a, b) and (b, a), and a zero partial changes nothing, so
// up to four partials are (0 + 2) + (1 + 3).  (One thread adding the partials
// in order took 11.3 us for 717 records of 16.)
__device__ inline void merge_sums(double& s, double& c, double s2, double c2) {
    double t, e;
    two_sum(s, s2, t, e);
    s = t;
    c = (c + c2) + e;
}

__device__ inline void partial_merge(TilePartial& a, const TilePartial& b) {
    a.A += b.A;
    a.B += b.B;
    merge_sums(a.s, a.sc, b.s, b.sc);
    merge_sums(a.q, a.qc, b.q, b.qc);
    a.maxbits = max(a.maxbits, b.maxbits);
    a.nan_count += b.nan_count;
    a.inf_count += b.inf_count;
}

__device__ inline TilePartial no_partial() { return TilePartial{0, 0, 0.0, 0.0, 0.0, 0.0, 0u, 0u, 0u, 0u}; }

// By one thread, nt <= 4.
constexpr int kThreadCombine = 4;
__device__ inline TilePartial combine_few(const TilePartial* pp, int nt) {
    TilePartial p[kThreadCombine];
#pragma unroll
    for (int i = 0; i < kThreadCombine; ++i) p[i] = i < nt ? pp[i] : no_partial();
    partial_merge(p[0], p[2]);
    partial_merge(p[1], p[3]);
    partial_merge(p[0], p[1]);
    return p[0];
}

template <int M>
__device__ inline double row_lane_f64(double v) {
    double r;
    from_bits(row_xor_u64<M>(bits_of(v)), r);
    return r;
}
template <int M>
__device__ inline void merge_level(TilePartial& p) {
    TilePartial o;
    o.A = row_xor_u64<M>(p.A);
    o.B = row_xor_u64<M>(p.B);
    o.s = row_lane_f64<M>(p.s);
    o.sc = row_lane_f64<M>(p.sc);
    o.q = row_lane_f64<M>(p.q);
    o.qc = row_lane_f64<M>(p.qc);
    o.maxbits = row_xor_u32<M>(p.maxbits);
    o.nan_count = row_xor_u32<M>(p.nan_count);
    o.inf_count = row_xor_u32<M>(p.inf_count);
    partial_merge(p, o);
}

// By sixteen lanes of a row, all of them active; every lane gets the result.
__device__ inline TilePartial combine_row(const TilePartial* pp, int64_t nt, int l) {
    TilePartial p = l < nt ? pp[l] : no_partial();
    // the rest in batches, so that a batch's loads are in flight together
    constexpr int kBatch = 3;
    for (int64_t x0 = l + 16; x0 < nt; x0 += 16 * kBatch) {
        TilePartial q[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) q[i] = x0 + 16 * i < nt ? pp[x0 + 16 * i] : no_partial();
#pragma unroll
        for (int i = 0; i < kBatch; ++i) partial_merge(p, q[i]);
    }
    merge_level<8>(p);
    merge_level<4>(p);
    merge_level<2>(p);
    merge_level<1>(p);
    return p;
}

__device__ inline double maxbits_to_f64(uint32_t bits, int dtype) {
    if (dtype == C3_F32) return (double)__uint_as_float(bits);
    if (dtype == C3_BF16) return (double)__uint_as_float(bits << 16);
    if (dtype == C3_F16) return f16_to_f64(bits);
    return 0.0;
}

// ti by value: the tensor's description in one batch of loads, so that the
// chain over the dimensions runs on registers instead of waiting for each in
// turn.
__device__ inline void write_record(c3_chunk_record_t* rec, const TensorInfo ti, int t, uint64_t k,
                                    uint64_t n, const TilePartial& p) {
    const int dtype = ti.dtype, ndim = ti.ndim;
    uint64_t h = fmix64(kTag ^ ((uint64_t)(uint32_t)dtype << 32) ^ (uint64_t)(uint32_t)ndim);
#pragma unroll
    for (int d = 0; d < C3_MAX_NDIM; ++d)
        if (d < ndim) h = fmix64(h ^ (uint64_t)ti.shape[d]);
    h = fmix64(h ^ k);
    h = fmix64(h ^ n);
    h = fmix64(h ^ p.A);
    h = fmix64(h ^ p.B);
    const uint64_t es = dtype == C3_F32 ? 4 : (dtype == C3_RAW ? 1 : 2);
    rec->sig = h;
    rec->n_elems = n / es;
    rec->nan_count = p.nan_count;
    rec->inf_count = p.inf_count;
    rec->tensor = (uint32_t)t;
    rec->chunk_in_tensor = (uint32_t)k;
    rec->absmax = maxbits_to_f64(p.maxbits, dtype);
    rec->sum = p.s + p.sc;
    rec->sumsq = p.q + p.qc;
    rec->reserved = 0;
}

}  // namespace c3
