// Device-side description of a K = T reduction and the scalar functions of the gate's stores (gfx950).
#pragma once

#include "ssm_internal.h"

namespace ssm {

typedef float v16f __attribute__((ext_vector_type(16)));

struct GemmDev {
    const float *A; long lda;
    const float *B; long ldb;
    float *C; long ldc;
    int M, N, K, kper;      // kper: K range per split (multiple of the K tile)
    int ntm, ntn;
    // placement of the (tile, split) work items on the 8 XCDs: slots per XCD, mapping mode and its
    // parameter, first slot of this problem in its launch
    int splits, nx, mode, par, slot0;
    FastDiv by_ntn, by_par;
    AbsMax amaxA, amaxB;    // two-plane fp16 staging only
};

__device__ __forceinline__ float gelu_derivative(float x)
{
    // d/dx [x Phi(x)] = Phi(x) + x phi(x)
    const float cdf = 0.5f * erfcf(-0.70710678118654752f * x);
    const float pdf = 0.39894228040143268f * __expf(-0.5f * x * x);
    return fmaf(x, pdf, cdf);
}
__device__ __forceinline__ float gelu_value(float x)
{
    // x Phi(x) with Phi(x) = erfc(-x / sqrt 2) / 2 (no cancellation in the lower tail)
    return 0.5f * x * erfcf(-0.70710678118654752f * x);
}
__device__ __forceinline__ float sigmoidf(float z)
{
    // e^-|z| never overflows; both branches are exact rewrites of 1 / (1 + e^-z)
    const float e = __expf(-fabsf(z));
    const float r = 1.f / (1.f + e);
    return z >= 0.f ? r : e * r;
}

}  // namespace ssm
