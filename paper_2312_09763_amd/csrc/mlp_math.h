// Device arithmetic shared by the learned beam's training and inference kernels.
#pragma once

#include "mlp.h"

namespace mv {
namespace mlp {

__device__ inline float silu(float z) { return z / (1.0f + __expf(-z)); }

// dL/dz from dL/dh: dh * d SiLU/dz = dh * s (1 + z (1 - s)),  s = 1 / (1 + exp(-z))
__device__ inline float silu_grad(float dh, float z) {
    const float s = 1.0f / (1.0f + __expf(-z));
    return dh * s * (1.0f + z * (1.0f - s));
}

// sin / cos of 2 pi r with the hardware units (argument in revolutions) after reduction
__device__ inline void sincos_rev(float r, float &s, float &c) {
    r -= rintf(r);
    s = __builtin_amdgcn_sinf(r);
    c = __builtin_amdgcn_cosf(r);
}

// T_0..T_{kBasis-1} of the first kind at t (three-term recurrence)
__device__ inline void chebyshev(float t, float (&T)[kBasis]) {
    T[0] = 1.0f;
    T[1] = t;
#pragma unroll
    for (int k = 2; k < kBasis; k++) T[k] = 2.0f * t * T[k - 1] - T[k - 2];
}

// Adam (Kingma & Ba 2015) on one parameter.
__device__ inline float adam_step(float p, float g, float &m1, float &m2, int64_t step, float lr, float b1, float b2,
                                  float eps) {
    const float a = b1 * m1 + (1.0f - b1) * g;
    const float b = b2 * m2 + (1.0f - b2) * g * g;
    m1 = a;
    m2 = b;
    const float ah = a / (1.0f - powf(b1, (float)step));
    const float bh = b / (1.0f - powf(b2, (float)step));
    return p - lr * ah / (sqrtf(bh) + eps);
}

}  // namespace mlp
}  // namespace mv
