// Optimizer-boundary check of C3 for gfx950 (Sec. 9; Sec. 6.2, the optimizer
// recipe): replay one AdamW step on a slice of every replica's state and sign
// the four input and three updated slices, in one pass over the inputs.
//
// One workgroup takes one tile of the slice of one replica.  Its four waves
// take the tile's 1 KiB blocks round-robin; a lane loads 16 bytes of each of
// the four tensors, replays its four elements, stores the three updated
// quadruples and folds all seven words into the accumulators of the seven
// tensors, whose partials the workgroup writes: the fold of signature_kernel
// (same quarters, same order, same bits) with the updated slices signed from
// registers.  A second launch, one workgroup, combines the partials, votes and
// writes the lists (c3_tail.h).
//
// Latency-bound: 8 replicas x 65,536 elements are 14.7 MB of traffic, 2 us,
// and the chain launch - loads - replay (two IEEE divisions and a square root
// an element) - reduction is what it costs.  Everything the kernel needs
// comes as arguments, so no plan is staged or read.  The replay and the
// signature as two launches, with the staged plan copied by the first and
// read by the second, took 6.0 + 7.7 us before the tail, and signed the
// inputs from a second read.
//
// The tile: smaller ones give more workgroups, whose waves replay fewer blocks
// one after the other, and more partials to combine.  us per check by tile:
//                  2      4      8     16     32     64 KiB
//   2 x  64 KiB  10.6   10.5   11.2
//   2 x 256 KiB  12.4   11.4   12.0   13.2   16.8
//   2 x   1 MiB  21.1   15.2   13.8   14.3   17.8   25.3
//   4 x 512 KiB  21.0   15.5   13.1   14.2   17.9   25.5
//   8 x 256 KiB  21.3   15.1   13.7   14.6   18.4
//   8 x   1 MiB  59.3   36.7   27.7   22.5   23.2   29.0
//   8 x   4 MiB                76.3   58.3   54.1   49.8
// so by default about 256 workgroups, or 32 a replica for eight and more
// (c3_api.cpp).  Tiles need not divide the slice: powers of two that do, of 1 KiB
// for a slice of an odd number of KiB, take 33.9 us for 8 x 257 KiB and 203 for
// 8 x 2,047 KiB, whole KiB 13.9 and 34.8.  (Three launches took 20.7 us for 8 x
// 256 KiB and 91 for 16 x 2 MiB, where these two take 13.9 and 50.9.)
#include "c3_adamw_step.h"
#include "c3_device.h"
#include "c3_fold.h"
#include "c3_internal.h"
#include "c3_tail.h"

namespace c3 {

constexpr int kOptThreads = 256;
constexpr int kOptSlices = 7;       // param, grad, exp_avg, exp_avg_sq, then the updated three
constexpr int kOptUnroll = 2;       // blocks in flight per wave
static_assert(kFoldBlocks % kOptUnroll == 0, "folds at the end of a batch");

struct OptBlock {
    float4 x[4];
};

__device__ __forceinline__ u32x4 words_of(float4 v) {
    u32x4 w;
    w.x = __float_as_uint(v.x);
    w.y = __float_as_uint(v.y);
    w.z = __float_as_uint(v.z);
    w.w = __float_as_uint(v.w);
    return w;
}

// Four elements of one tensor, of which `valid` exist; the rest read as zero
// bytes, as the signature pads them.
__device__ __forceinline__ float4 load_quad(const float* p, int valid) {
    if (valid >= 4) return *reinterpret_cast<const float4*>(p);
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (valid > 0) v.x = p[0];
    if (valid > 1) v.y = p[1];
    if (valid > 2) v.z = p[2];
    return v;
}
__device__ __forceinline__ void store_quad(float* p, float4 v, int valid) {
    if (valid >= 4) {
        *reinterpret_cast<float4*>(p) = v;
        return;
    }
    if (valid > 0) p[0] = v.x;
    if (valid > 1) p[1] = v.y;
    if (valid > 2) p[2] = v.z;
}

// The seven words of a lane's quad; elements past the slice are zero in all.
__device__ __forceinline__ void replay_quad(const AdamwConst& c, const OptBlock& b, int valid,
                                            float4 (&y)[3]) {
    const float4 p = b.x[0], g = b.x[1], m = b.x[2], v = b.x[3];
    const Upd u0 = adamw_one(c, p.x, g.x, m.x, v.x);
    const Upd u1 = adamw_one(c, p.y, g.y, m.y, v.y);
    const Upd u2 = adamw_one(c, p.z, g.z, m.z, v.z);
    const Upd u3 = adamw_one(c, p.w, g.w, m.w, v.w);
    y[0] = make_float4(u0.p, u1.p, u2.p, u3.p);
    y[1] = make_float4(u0.m, u1.m, u2.m, u3.m);
    y[2] = make_float4(u0.v, u1.v, u2.v, u3.v);
    if (valid < 4) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            y[j].w = 0.0f;
            if (valid < 3) y[j].z = 0.0f;
            if (valid < 2) y[j].y = 0.0f;
        }
    }
}

// blocks: 1 KiB blocks (256 elements) per tile; partials [R][7][gridDim.x].
// Every base is 16-byte aligned, offset and stride are multiples of 256.
// FOLD: tiles of more than 4 kFoldBlocks blocks that do not divide the slice as
// a power of two, whose sums of squares are folded on the way (LaneSums); 224
// registers, two waves a SIMD for three.
template <bool FOLD>
__global__ void __launch_bounds__(kOptThreads) optimizer_slices_kernel(
    AdamwPtrs ptrs, AdamwConst c, int64_t offset, int64_t n, int blocks, float* __restrict__ out,
    int64_t stride, TilePartial* __restrict__ partials) {
    __shared__ TilePartial lds[kOptThreads / 64][kOptSlices];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = blockIdx.y;
    const float* in[4] = {ptrs.param[r] + offset, ptrs.grad[r] + offset, ptrs.exp_avg[r] + offset,
                          ptrs.exp_avg_sq[r] + offset};
    float* const o = out + (int64_t)r * 3 * stride;
    const int64_t blk0 = (int64_t)blockIdx.x * blocks;        // of the slice: one chunk
    // this tile's blocks that hold elements
    const int64_t left = (n + 255) / 256 - blk0;
    const int nblk = left < blocks ? (int)left : blocks;
    const LaneKeys K = lane_keys(lane);

    LaneFold<1> f[kOptSlices];
    LaneSums<C3_F32, FOLD> sums[kOptSlices];
    float mf[kOptSlices];
#pragma unroll
    for (int t = 0; t < kOptSlices; ++t) {
        f[t].A = f[t].B = 0;
        f[t].mx = f[t].nan_c = f[t].inf_c = 0u;
        mf[t] = 0.0f;
    }
    auto at = [&](int k) { return (blk0 + k) * 256 + lane * 4; };
    auto valid_of = [&](int64_t e) { return n - e >= 4 ? 4 : n > e ? (int)(n - e) : 0; };
    auto fold = [&](const OptBlock& b, const float4 (&y)[3], uint32_t beta) {
#pragma unroll
        for (int t = 0; t < kOptSlices; ++t) {
            const u32x4 w = words_of(t < 4 ? b.x[t & 3] : y[t < 4 ? 0 : t - 4]);
            nh16(w, K, beta, f[t].A, f[t].B);
            stats_fast<C3_F32>(w, sums[t], mf[t]);
        }
    };
    // block k of the tile is block k / 4 of its quarter
    auto fold_sums = [&](int k) {
        if (!FOLD || (k >> 2) % kFoldBlocks != kFoldBlocks - 1) return;
#pragma unroll
        for (int t = 0; t < kOptSlices; ++t) sums[t].fold();
    };
    auto take_sums = [&](int t) {
        f[t].s[0] = sums[t].s;
        f[t].q[0] = sums[t].squares();
    };
    // whole blocks without a test per lane; the slice's last one may be partial
    const int nwhole = (int)min((int64_t)nblk, n / 256 - blk0);
    for (int k0 = wave; k0 < nwhole; k0 += 4 * kOptUnroll) {
        OptBlock b[kOptUnroll];
#pragma unroll
        for (int u = 0; u < kOptUnroll; ++u)
            if (k0 + 4 * u < nwhole) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    b[u].x[t] = *reinterpret_cast<const float4*>(in[t] + at(k0 + 4 * u));
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kOptUnroll; ++u) {
            const int k = k0 + 4 * u;
            if (k >= nwhole) break;
            float4 y[3];
            replay_quad(c, b[u], 4, y);
#pragma unroll
            for (int j = 0; j < 3; ++j) *reinterpret_cast<float4*>(o + j * stride + at(k)) = y[j];
            fold(b[u], y, block_beta((uint32_t)(blk0 + k)));
        }
        // (k0 - wave) / 4 is even: the second block of a batch may be the last of four
        if (k0 + 4 * (kOptUnroll - 1) < nwhole) fold_sums(k0 + 4 * (kOptUnroll - 1));
    }
    if (nwhole < nblk && (nwhole & 3) == wave) {
        const int64_t e = at(nwhole);
        const int valid = valid_of(e);
        if (valid > 0) {
            OptBlock b;
            float4 y[3];
#pragma unroll
            for (int t = 0; t < 4; ++t) b.x[t] = load_quad(in[t] + e, valid);
            replay_quad(c, b, valid, y);
#pragma unroll
            for (int j = 0; j < 3; ++j) store_quad(o + j * stride + e, y[j], valid);
            fold(b, y, block_beta((uint32_t)(blk0 + nwhole)));
        }
    }
    // a lane that met a NaN or Inf replays its elements once more, classifying
    // (in all seven slices: the finite ones come out as they were)
    bool finite = true;
#pragma unroll
    for (int t = 0; t < kOptSlices; ++t) {
        take_sums(t);
        finite = finite && __builtin_isfinite(f[t].s[0]) && __builtin_isfinite(f[t].q[0]);
        f[t].mx = magnitude_bits<C3_F32>(mf[t]);
    }
    if (!finite) {
#pragma unroll
        for (int t = 0; t < kOptSlices; ++t) {
            sums[t] = LaneSums<C3_F32, FOLD>();
            f[t].mx = 0u;
        }
        for (int k = wave; k < nblk; k += 4) {
            const int64_t e = at(k);
            const int valid = valid_of(e);
            if (valid <= 0) break;
            OptBlock b;
            float4 y[3];
#pragma unroll
            for (int t = 0; t < 4; ++t) b.x[t] = load_quad(in[t] + e, valid);
            replay_quad(c, b, valid, y);
#pragma unroll
            for (int t = 0; t < kOptSlices; ++t)
                stats_slow<C3_F32>(words_of(t < 4 ? b.x[t & 3] : y[t < 4 ? 0 : t - 4]), sums[t], f[t].mx,
                                   f[t].nan_c, f[t].inf_c);
            if (k < nwhole) fold_sums(k);
        }
#pragma unroll
        for (int t = 0; t < kOptSlices; ++t) take_sums(t);
    }
    // wave_reduce of two slices at a time: after the level of 32 the lower and
    // upper lanes hold A and B (sum and sum of squares), after that of 16 the
    // even and odd rows the first and second slice
#pragma unroll
    for (int t = 0; t < kOptSlices; t += 2) {
        const int t2 = t + 1 < kOptSlices ? t + 1 : t;
        const uint64_t ab = row_sum(fold16(fold32(f[t].A, f[t].B), fold32(f[t2].A, f[t2].B)));
        const double sq = row_sum(fold16(fold32(f[t].s[0], f[t].q[0]), fold32(f[t2].s[0], f[t2].q[0])));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (t + i >= kOptSlices) break;
            TilePartial p;
            p.A = readlane_u64(ab, 16 * i);
            p.B = readlane_u64(ab, 32 + 16 * i);
            from_bits(readlane_u64(bits_of(sq), 16 * i), p.s);
            from_bits(readlane_u64(bits_of(sq), 32 + 16 * i), p.q);
            p.sc = p.qc = 0.0;
            reduce_counts(p, f[t + i].mx, f[t + i].nan_c, f[t + i].inf_c);
            if (lane == 0) lds[wave][t + i] = p;
        }
    }
    __syncthreads();
    if (threadIdx.x < kOptSlices) {
        const int t = threadIdx.x;
        TilePartial p = lds[0][t];
#pragma unroll
        for (int w = 1; w < kOptThreads / 64; ++w) partial_add(p, lds[w][t]);
        partials[((int64_t)r * kOptSlices + t) * gridDim.x + blockIdx.x] = p;
    }
}

// Records of the R x 7 slices from nt partials each, votes and lists.
__global__ void __launch_bounds__(kTailThreads) optimizer_tail_kernel(
    const TilePartial* __restrict__ partials, int64_t nt, int64_t n, int R,
    c3_chunk_record_t* __restrict__ records, TailOut out) {
    __shared__ c3_chunk_record_t rec[kOptSlices * C3_MAX_REPLICAS];
    const int l = threadIdx.x & 15;
    for (int i = threadIdx.x >> 4; i < R * kOptSlices; i += kTailThreads / 16) {
        const TilePartial p = combine_row(partials + i * nt, nt, l);
        if (l == 0) {
            TensorInfo ti = {};
            ti.nbytes = (uint64_t)n * 4;
            ti.dtype = C3_F32;
            ti.ndim = 1;
            ti.shape[0] = n;
            write_record(&rec[i], ti, i % kOptSlices, 0, ti.nbytes, p);
            records[i] = rec[i];
        }
    }
    tail_votes_and_lists(rec, R, kOptSlices, out);
}

int64_t optimizer_tiles(int64_t n, uint64_t tile_bytes) {
    return ((int64_t)(n * 4) + (int64_t)tile_bytes - 1) / (int64_t)tile_bytes;
}

uint64_t optimizer_partials_bytes(int R, int64_t slice_elems, uint64_t tile_bytes) {
    return (uint64_t)R * kOptSlices * (uint64_t)optimizer_tiles(slice_elems, tile_bytes) * sizeof(TilePartial);
}

hipError_t launch_optimizer_check(const AdamwPtrs& ptrs, const AdamwConst& c, int R, int64_t offset,
                                  int64_t n, uint64_t tile_bytes, float* updated, int64_t stride,
                                  void* partials, c3_chunk_record_t* records, const TailOut& out,
                                  hipStream_t stream) {
    const int64_t nt = optimizer_tiles(n, tile_bytes);
    TilePartial* pp = static_cast<TilePartial*>(partials);
    if (nt > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int blocks = (int)(tile_bytes / 1024);
    const bool folds = blocks > 4 * kFoldBlocks && folded_tiles((uint64_t)stride * 4, tile_bytes);
    hipLaunchKernelGGL(folds ? optimizer_slices_kernel<true> : optimizer_slices_kernel<false>,
                       dim3((unsigned)nt, (unsigned)R), dim3(kOptThreads), 0, stream, ptrs, c, offset, n,
                       blocks, updated, stride, pp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(optimizer_tail_kernel, dim3(1), dim3(kTailThreads), 0, stream, pp, nt, n, R,
                       records, out);
    return hipGetLastError();
}

}  // namespace c3
