// Receiver sampling and DTFT arithmetic shared by the kernels that do it
// inside the stencil launches and those that do it after a whole time loop:
// one text, so that both round alike.
#pragma once

#include "emm_internal.h"

namespace emm {

// u = sum over the (2r)^3 tensor-product stencil of w * F(q), reduced in FP64
// over the wavefront; F(q) is the field value under stencil point q.
template <int R, typename Value>
__device__ __forceinline__ double rec_sum(const float *w, int lane, Value F) {
    constexpr int L = 2 * R;
    double u = 0.0;
    for (int q = lane; q < L * L * L; q += 64) {
        const int a = q % L, b = (q / L) % L, c = q / (L * L);
        const float wt = w[a] * w[L + b] * w[2 * L + c];
        u += (double)wt * (double)F(q, a, b, c);
    }
    for (int off = 32; off > 0; off >>= 1) u += __shfl_xor(u, off, 64);
    return u;
}

// acc += u exp(i w' t) in FP64
__device__ __forceinline__ void rec_add(double2 &a, double u, double2 ph) {
    a.x += u * ph.x;
    a.y += u * ph.y;
}

// the same as an FP32 Kahan-compensated sum: (re, c_re, im, c_im)
__device__ __forceinline__ void rec_add(float4 &a, double u, double2 ph) {
    const float uf = (float)u;
    const float xr = uf * (float)ph.x, xi = uf * (float)ph.y;
    float y = xr - a.y, t = a.x + y;
    a.y = (t - a.x) - y;
    a.x = t;
    y = xi - a.w;
    t = a.z + y;
    a.w = (t - a.z) - y;
    a.z = t;
}

}  // namespace emm
