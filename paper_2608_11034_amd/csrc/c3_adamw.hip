// Optimizer-boundary replay of C3 for gfx950 (Sec. 9, optimizer boundary;
// Sec. 6.2, the optimizer recipe): one AdamW step re-applied to the slice
// [offset, offset + n) of each of R replicas' fp32 parameter, gradient and
// moment tensors, written out as updated (parameter, first moment, second
// moment) slices for the signature pass to compare across replicas.  The
// replicas' own tensors are not modified.
//
// The update is AdamW with decoupled weight decay in the operation order of
// PyTorch's single-tensor AdamW (amsgrad off, not maximizing), each fp32
// operation rounded once, no contraction, IEEE division and square root:
//     p1 = p * decay                       decay = fp32(1 - lr wd)
//     m1 = m + w (g - m)          if |w| < 1/2, w = fp32(1 - beta1)
//        = g - (g - m) (1 - w)    otherwise
//     v1 = v * beta2 + (c2 g) g            c2 = fp32(1 - beta2)
//     d  = sqrt(v1) / s2 + eps             s2 = fp32(sqrt(1 - beta2^t))
//     p2 = p1 + (-a) (m1 / d)              a  = fp32(lr / (1 - beta1^t))
// NaN results are stored as the default quiet NaN 0x7FC00000, so the bytes
// that the signature pass hashes do not depend on how an implementation
// propagates NaN payloads.
//
// Memory: the kernel reads 16 B and writes 12 B per (element, replica).
// Output row (replica r, tensor j) starts at out + (3 r + j) * stride.
// Each thread handles four consecutive elements of one replica with 128-bit
// loads and stores when every base pointer, the offset and n allow it
// (4-element aligned), else one element with 32-bit accesses; grid.y is
// the replica.  (128-bit accesses at 4-byte alignment were slower than 32-bit
// ones: 2 replicas x 16,777,215 elements 167.9 against 166.4 us.)
#include "c3_adamw_step.h"
#include "c3_internal.h"

namespace c3 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// A replay that moves more than the 256 MB memory-side cache holds streams
// past the caches: the inputs are read once and the updates not read by this
// kernel.  us per call, plain / non-temporal loads / loads and stores: 2 replicas
// x 16.8M elements (940 MB) 178.7 / 172.5 / 160.3, on three sets of buffers in
// turn 172 / 169 / 163; 8 x 4.0M 163.4 / 159.2 / 146.9; 2 x 6.0M (336 MB) 61.3 / 58.9
// / 54.3.  (Two quads a thread were 3% slower than one.)  Smaller replays keep
// their updates cached for the signature that follows.
constexpr int64_t kStreamBytes = 256 << 20;

template <bool NT>
__device__ __forceinline__ f32x4 load_quad(const float* p) {
    const f32x4* q = reinterpret_cast<const f32x4*>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}
template <bool NT>
__device__ __forceinline__ void store_quad(float* p, f32x4 v) {
    f32x4* q = reinterpret_cast<f32x4*>(p);
    if constexpr (NT) __builtin_nontemporal_store(v, q);
    else *q = v;
}

// Four elements a thread.  n, offset and stride are multiples of 4 and every
// base is 16-byte aligned.
template <bool NT>
__global__ void __launch_bounds__(256) adamw_slice_vec4_kernel(AdamwPtrs ptrs, AdamwConst c,
                                                               int64_t offset, int64_t n,
                                                               float* __restrict__ out,
                                                               int64_t stride) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    const int r = blockIdx.y;
    if (i >= n) return;
    const int64_t e = offset + i;
    f32x4 x[4], y[3];
    x[0] = load_quad<NT>(ptrs.param[r] + e);
    x[1] = load_quad<NT>(ptrs.grad[r] + e);
    x[2] = load_quad<NT>(ptrs.exp_avg[r] + e);
    x[3] = load_quad<NT>(ptrs.exp_avg_sq[r] + e);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const Upd u = adamw_one(c, x[0][j], x[1][j], x[2][j], x[3][j]);
        y[0][j] = u.p;
        y[1][j] = u.m;
        y[2][j] = u.v;
    }
    float* const o = out + (int64_t)r * 3 * stride + i;
#pragma unroll
    for (int t = 0; t < 3; ++t) store_quad<NT>(o + t * stride, y[t]);
}

// One element a thread: any offset, length, stride and alignment.  (Rows of
// odd stride: non-temporal accesses gain 3% at 2 x 16,777,215 elements and lose
// 6% at 8 x 4,000,001, so none here.)
__global__ void __launch_bounds__(256) adamw_slice_kernel(AdamwPtrs ptrs, AdamwConst c,
                                                          int64_t offset, int64_t n,
                                                          float* __restrict__ out, int64_t stride) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= n) return;
    const int64_t e = offset + i;
    const Upd u = adamw_one(c, ptrs.param[r][e], ptrs.grad[r][e], ptrs.exp_avg[r][e],
                            ptrs.exp_avg_sq[r][e]);
    float* o = out + (int64_t)r * 3 * stride;
    o[i] = u.p;
    o[stride + i] = u.m;
    o[2 * stride + i] = u.v;
}

hipError_t launch_adamw_slice(const AdamwPtrs& ptrs, const AdamwConst& c, int R, bool vec4,
                              int64_t offset, int64_t n, float* out, int64_t stride,
                              hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int64_t threads = vec4 ? n / 4 : n;
    const int64_t blocks = (threads + 255) / 256;
    if (blocks > 0x7FFFFFFF || R > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks, (unsigned)R), block(256);
    const bool nt = n * R * 28 > kStreamBytes;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, ptrs, c, offset, n, out, stride);
    };
    if (vec4) nt ? launch(adamw_slice_vec4_kernel<true>) : launch(adamw_slice_vec4_kernel<false>);
    else launch(adamw_slice_kernel);
    return hipGetLastError();
}

}  // namespace c3
