// Device-side building blocks of the C3 kernels: the C3SIG-1 primitives
// (SplitMix64 key stream, fmix64 finalizer), wave64 reductions and
// error-free fp64 addition.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace c3 {

// C3SIG-1 constants: key-stream seed, finalize domain tag, block multiplier.
constexpr uint64_t kKeySeed = 0x43335349472D3101ull;
constexpr uint64_t kTag = 0x4333534947310001ull;
constexpr uint32_t kBlockMul = 0x9E3779B9u;
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

// i-th output (0-based) of SplitMix64 started at `seed`: the generator adds
// gamma before each output, so output i mixes seed + (i + 1) * gamma.
__device__ __host__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * kGamma;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline uint32_t nh_key(uint32_t i) { return (uint32_t)splitmix64_at(kKeySeed, i); }

// MurmurHash3's 64-bit finalizer.
__device__ __host__ inline uint64_t fmix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xFF51AFD7ED558CCDull;
    k ^= k >> 33;
    k *= 0xC4CEB9FE1A85EC53ull;
    k ^= k >> 33;
    return k;
}

// Knuth's TwoSum: s + e == a + b exactly, s = fl(a + b).  Requires that the
// compiler does not reassociate (no fast-math).
__device__ inline void two_sum(double a, double b, double& s, double& e) {
    s = a + b;
    double bb = s - a;
    double aa = s - bb;
    e = (a - aa) + (b - bb);
}

// (s, c) += (s2, c2) with the rounding error of s + s2 carried in c.
__device__ inline void comp_add(double& s, double& c, double s2, double c2) {
    double t, e;
    two_sum(s, s2, t, e);
    s = t;
    c = c + (c2 + e);
}

// ---------------------------------------------------------------------------
// wave64 cross-lane helpers (ds_bpermute, DPP and lane swaps)
// ---------------------------------------------------------------------------
__device__ inline uint32_t shfl_xor_u32(uint32_t v, int m) {
    return (uint32_t)__shfl_xor((int)v, m, 64);
}
__device__ inline uint64_t shfl_xor_u64(uint64_t v, int m) {
    uint32_t lo = shfl_xor_u32((uint32_t)v, m), hi = shfl_xor_u32((uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t shfl_u64(uint64_t v, int src) {
    uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
    uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64);
    return ((uint64_t)hi << 32) | lo;
}

__device__ inline uint64_t ballot64(bool p) { return __ballot(p); }

// The value of the lane whose index differs in bit M (1, 2, 4 or 8), by DPP
// moves inside a row of 16: no LDS round trip.
template <int M>
__device__ __forceinline__ uint32_t row_xor_u32(uint32_t v) {
    const int iv = (int)v;
    if constexpr (M == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0xB1, 0xF, 0xF, false);
    else if constexpr (M == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x4E, 0xF, 0xF, false);
    else if constexpr (M == 4)      // mirror of 8 lanes (^7), then of 4 (^3)
        return (uint32_t)__builtin_amdgcn_mov_dpp(
            __builtin_amdgcn_mov_dpp(iv, 0x141, 0xF, 0xF, false), 0x1B, 0xF, 0xF, false);
    else return (uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x128, 0xF, 0xF, false);   // rotate by 8
}
template <int M>
__device__ __forceinline__ uint64_t row_xor_u64(uint64_t v) {
    return ((uint64_t)row_xor_u32<M>((uint32_t)(v >> 32)) << 32) | row_xor_u32<M>((uint32_t)v);
}

__device__ __forceinline__ uint64_t bits_of(double v) { return (uint64_t)__double_as_longlong(v); }
__device__ __forceinline__ uint64_t bits_of(uint64_t v) { return v; }
__device__ __forceinline__ void from_bits(uint64_t b, double& v) { v = __longlong_as_double((long long)b); }
__device__ __forceinline__ void from_bits(uint64_t b, uint64_t& v) { v = b; }

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// One level of two reductions at once.  fold32(a, b): the lower 32 lanes get
// a + (a of lane ^ 32), the upper ones the same of b; fold16(a, b): even rows
// of 16 lanes get a + (a of lane ^ 16), odd rows the same of b.  One swap per
// 32-bit word instead of a shuffle for each of the two values.
template <typename V>
__device__ __forceinline__ V fold32(V a, V b) {
    const uint64_t x = bits_of(a), y = bits_of(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    V p, q;
    from_bits(((uint64_t)hi[0] << 32) | lo[0], p);
    from_bits(((uint64_t)hi[1] << 32) | lo[1], q);
    return p + q;
}
template <typename V>
__device__ __forceinline__ V fold16(V a, V b) {
    const uint64_t x = bits_of(a), y = bits_of(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    V p, q;
    from_bits(((uint64_t)hi[0] << 32) | lo[0], p);
    from_bits(((uint64_t)hi[1] << 32) | lo[1], q);
    return p + q;
}
// The remaining levels, 8 to 1: every lane gets its row's sum.
template <int M, typename V>
__device__ __forceinline__ V row_add(V a) {
    V b;
    from_bits(row_xor_u64<M>(bits_of(a)), b);
    return a + b;
}
template <typename V>
__device__ __forceinline__ V row_sum(V a) {
    return row_add<1>(row_add<2>(row_add<4>(row_add<8>(a))));
}
// Maximum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max(b[0], b[1]);
    v = max(v, row_xor_u32<8>(v));
    v = max(v, row_xor_u32<4>(v));
    v = max(v, row_xor_u32<2>(v));
    return max(v, row_xor_u32<1>(v));
}

// Orders a wave's own LDS accesses (LDS instructions of one wave execute in
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// 128-bit streaming loads
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4 gu32x4;

// 128-bit streaming load from global memory, non-temporal (read once).
__device__ inline u32x4 load16(const u32x4* p) {
    return __builtin_nontemporal_load((gu32x4*)p);
}

// Raw buffer resource over the `len` bytes at `base` (stride 0, untyped
// 32-bit data format in the descriptor's last word, as gfx9 buffer loads
// require).  Callers load only whole 16-byte segments of whole 1 KiB blocks
// that lie inside `len`, so nothing depends on the hardware range check.
// Tiles are at most 16 MiB, so `len` fits the 32-bit record count.  Base and
// length are taken from the first lane: the resource must sit in scalar
// registers even when the compiler cannot prove them uniform.
constexpr int kRawBufferWord3 = 0x00020000;

__device__ inline __amdgpu_buffer_rsrc_t tile_resource(const uint8_t* base, uint32_t len) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const int n = __builtin_amdgcn_readfirstlane((int)len);
    void* b = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(b, (short)0, n, kRawBufferWord3);
}

// 128-bit non-temporal buffer load at voffset + soffset bytes.
__device__ inline u32x4 load16_buf(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
    constexpr int kNonTemporal = 2;
    return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, kNonTemporal);
}

}  // namespace c3
