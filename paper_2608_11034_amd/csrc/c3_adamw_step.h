// One element of the AdamW step of c3_adamw.hip (its operation order and
// roundings), shared with the optimizer-boundary kernel.
#pragma once

#include "c3_internal.h"

namespace c3 {

__device__ __forceinline__ float canon_nan(float x) {
    return x != x ? __uint_as_float(0x7FC00000u) : x;
}

struct Upd {
    float p, m, v;
};

__device__ __forceinline__ Upd adamw_one(const AdamwConst& c, float p, float g, float m, float v) {
    Upd u;
    const float p1 = p * c.decay;
    float m1;
    if (c.lerp_small) {
        m1 = m + c.w * (g - m);
    } else {
        m1 = g - (g - m) * c.one_minus_w;
    }
    const float v1 = v * c.beta2 + (c.c2 * g) * g;
    const float d = __builtin_sqrtf(v1) / c.s2 + c.eps;
    u.p = canon_nan(p1 + c.neg_step * (m1 / d));
    u.m = canon_nan(m1);
    u.v = canon_nan(v1);
    return u;
}

}  // namespace c3
