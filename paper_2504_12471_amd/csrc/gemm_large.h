// What the large bf16 products (kernels_gemm_mfma.hip, kernels_gemm_pair.hip, kernels_gemm_wgrad.hip) share.
#pragma once

#include "gemm_map.h"
#include "launch.h"

namespace d2ft {

// all but the N youngest of the wavefront's vector memory operations are complete (they complete in order)
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ---- GELU for the bf16 epilogues ----
// The epilogue of FC1 (and of its backward) evaluates Phi on 65536 elements per tile, which on the
// vector ALUs costs as much time as the tile's MFMAs if done with erff (a reciprocal, an
// exponential and a polynomial).  Here Phi(z) = 0.5 + z * Q(z^2) with Q a degree-8 polynomial fitted
// on |z| <= 4 (Chebyshev fit of (Phi(z) - 0.5) / z; max absolute error 3.3e-5 including the clamp
// of |z| to 4), i.e. more than an order of magnitude below bf16 resolution: 11 FMA-class
// instructions and no transcendental.  The forward epilogue also evaluates GELU'(z) = Phi(z) + z phi(z)
// (one exponential for the density) and saves it in place of z, so the backward epilogue is one
// multiplication per element.
__device__ __forceinline__ float phi_poly(float z) {
    const float zc = fminf(fmaxf(z, -4.0f), 4.0f);
    const float u = zc * zc;
    float q = 1.043768652e-10f;
    q = fmaf(q, u, -8.556765862e-09f);
    q = fmaf(q, u, 3.133464190e-07f);
    q = fmaf(q, u, -6.888049885e-06f);
    q = fmaf(q, u, 1.036909179e-04f);
    q = fmaf(q, u, -1.155711931e-03f);
    q = fmaf(q, u, 9.929860060e-03f);
    q = fmaf(q, u, -6.646679917e-02f);
    q = fmaf(q, u, 3.989401704e-01f);
    return fmaf(zc, q, 0.5f);
}

// v <- GELU(v), d <- GELU'(v) of 8 pre-activations
__device__ __forceinline__ void gelu_pair8(float (&v)[8], float (&d)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float z = v[i], ph = phi_poly(z);
        d[i] = fmaf(z * 0.39894228040143267794f, __builtin_amdgcn_exp2f(-0.72134752044448170368f * z * z), ph);
        v[i] = z * ph;
    }
}

}  // namespace d2ft
