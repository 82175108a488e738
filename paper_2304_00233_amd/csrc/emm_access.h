// Global memory access of the plane-marching kernels.
#pragma once

#include "emm_internal.h"

namespace emm {

template <bool ST, typename P>
__device__ __forceinline__ auto ld1(P p) {
    if constexpr (ST) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool ST>
__device__ __forceinline__ void st1(float *p, float v) {
    if constexpr (ST) __builtin_nontemporal_store(v, p);
    else *p = v;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Global accesses of the plane loop: (scalar 64-bit base of a plane) + (32-bit
// byte offset of the thread's column), the pair that one load or store
// instruction takes, so that a plane's accesses cost no vector arithmetic.
// keep_s / keep_v stop the compiler from folding a sum of scalars into the
// vector part and from widening a column offset ahead of the loop.
typedef __attribute__((address_space(1))) char gchar;
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) unsigned guint;
__device__ __forceinline__ gchar *keep_s(gchar *q) {
    asm("" : "+s"(q));
    return q;
}
__device__ __forceinline__ void keep_v(unsigned &off) { asm("" : "+v"(off)); }
template <bool ST>
__device__ __forceinline__ float ldp(const gchar *pl, unsigned off) {
    return ld1<ST>((const gfloat *)(pl + off));
}
template <bool ST>
__device__ __forceinline__ void stp(gchar *pl, unsigned off, float v) {
    if constexpr (ST) __builtin_nontemporal_store(v, (gfloat *)(pl + off));
    else *(gfloat *)(pl + off) = v;
}

}  // namespace emm
