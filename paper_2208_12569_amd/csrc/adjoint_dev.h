// What the two reverse kernels (adjoint.hip, adjoint_quad.hip) share.
#pragma once

#include <hip/hip_runtime.h>

namespace fq {
namespace adj {

// value and gradient (local coordinates) of P(u,v,w) in monomial form
template <typename T>
__device__ __forceinline__ void poly_grad(const T c[8], T u, T v, T w, T g[3])
{
    g[0] = c[1] + c[4] * v + c[5] * w + c[7] * v * w;
    g[1] = c[2] + c[4] * u + c[6] * w + c[7] * u * w;
    g[2] = c[3] + c[5] * u + c[6] * v + c[7] * u * v;
}

template <typename T> __device__ __forceinline__ T tri_w(int q, T u, T v, T w)
{
    return ((q & 1) ? u : T(1) - u) * ((q & 2) ? v : T(1) - v) * ((q & 4) ? w : T(1) - w);
}

// Captures the accepted step of a replayed trial.
struct Capture {
    int *axis;
    double *H;
    int *clamp;
    template <typename T> __device__ __forceinline__ void accepted(int a, T h, int cl) const
    {
        *axis = a;
        *H = (double)h;
        *clamp = cl;
    }
};

}  // namespace adj
}  // namespace fq
