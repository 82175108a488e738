// HIP kernels of the discrete adjoint of the time loop (reverse of one
// leap-frog step of Section 3.1 with the CPML recursion of Section 3.4).
//
// Adjoint variables: Et = (dt/eps) * Ebar (the E adjoint scaled by the
// per-cell coefficient) and Hb = Hbar.  Reverse of step n, in order:
//   1. reverse of the H update: Et += (dt/eps) dt/mu0 curlT(F(Hb)), with
//      the transposed D+ tables (their stencil has the D- shape);
//   2. receiver sources of the E channels (stamp (n+1) dt);
//   3. reverse of the E update: grad += Ebar (E^{n+1} - E^n) (summed as
//      Et (E^{n+1} - E^n) in FP32 over a few steps, then divided by dt/eps
//      and added to the FP64 gradient) and
//      Hb -= curlT(F(Et)), with the transposed D- tables (D+ shape);
//   4. receiver sources of the H channels (stamp (n+1/2) dt).
// The curl structure is the forward one (component 1 has y and z taps,
// component 2 x and z, component 3 x and y).  F is the reverse of the CPML
// recursion psi = b psi + a d, d~ = d + psi, applied to the inputs of every
// derivative inside its slab: psibar = b Q + v, Q = psibar, v~ = v + a psibar
// (Q carried backwards in time).  Because F of a tap depends on that tap's
// own memory variable, a slab-only kernel applies it first and writes the
// filtered values to slab arrays that the gather reads instead of the raw
// field.
#include "emm_adjoint.h"
#include "emm_access.h"

#include <algorithm>
#include <type_traits>

namespace emm {

constexpr int AT = 256;

// 2./4. receiver adjoint sources: one thread per target cell of the
// injection list (cells sorted, contributions in a fixed order, so the sum
// is deterministic).  dchi/du_n of item q = sum_f Re(A[q][f] ph[n][f]).
__device__ __forceinline__ void adj_inject(const InjectParams &p, int n, int t) {
    if (t >= p.ncells) return;
    float acc = 0.f;
    for (int e = p.row[t]; e < p.row[t + 1]; ++e) {
        const int q = p.item[e];
        double sb = 0.0;
        for (int f = 0; f < p.nf; ++f) {
            const double2 A = p.A[(long long)q * p.nf + f];
            const double2 z = p.phase[(long long)n * p.nf + f];
            sb += A.x * z.x - A.y * z.y;
        }
        acc += p.w[e] * (float)sb;
    }
    const long long g = p.cell[t];
    const int comp = p.comp[t];
    float *F = comp == 0 ? p.F1 : (comp == 1 ? p.F2 : p.F3);
    const long long mc = p.mcell[t];
    const float scale = p.scale_ce ? (comp == 0 ? p.ce1[mc] : (comp == 1 ? p.ce2[mc] : p.ce3[mc])) : 1.f;
    F[g] += scale * acc;
}

// 1. CPML reverse filter on the slab cells of the update set, for the six
// (input component, tap axis) pairs.  One thread per slab cell of one axis.
// REV_H = true: inputs Hb, half-node tables (reverse of the H update);
// REV_H = false: inputs Et, integer-node tables (reverse of the E update).
// The blocks past the first nfilter inject the receiver adjoint sources that
// come before this filter in the order of the steps: they go into the same
// field, but into interior cells, never the slabs', so both run in one launch
// (either alone takes 5-6 us on a small grid, mostly launch).
template <bool REV_H>
__global__ __launch_bounds__(AT) void adj_filter(const AdjParams p, int nfilter, const InjectParams q, int n) {
    if ((int)blockIdx.x >= nfilter) {
        adj_inject(q, n, (blockIdx.x - nfilter) * AT + threadIdx.x);
        return;
    }
    const long long t = (long long)blockIdx.x * AT + threadIdx.x;
    const int r = p.r, nb = p.nb, nb2 = 2 * p.nb;
    const long long nx = (long long)p.n3 * p.n2 * nb2, ny = (long long)p.n3 * nb2 * p.n1,
                    nz = (long long)nb2 * p.n2 * p.n1;
    const long long per_src = nx + ny + nz;
    if (t >= per_src * p.nsrc) return;
    const int s = (int)(t / per_src);
    long long u = t - (long long)s * per_src;
    int axis, i, j, k, si;
    if (u < nx) {
        axis = 0;
        si = (int)(u % nb2);
        u /= nb2;
        j = (int)(u % p.n2);
        k = (int)(u / p.n2);
        i = si < nb ? si : si + (p.n1 - nb2);
    } else if (u < nx + ny) {
        axis = 1;
        u -= nx;
        i = (int)(u % p.n1);
        u /= p.n1;
        si = (int)(u % nb2);
        k = (int)(u / nb2);
        j = si < nb ? si : si + (p.n2 - nb2);
    } else {
        axis = 2;
        u -= nx + ny;
        i = (int)(u % p.n1);
        u /= p.n1;
        j = (int)(u % p.n2);
        si = (int)(u / p.n2);
        k = si < nb ? si : si + (p.n3 - nb2);
    }
    if (i < r || i > p.n1 - 1 - r || j < r || j > p.n2 - 1 - r || k < r || k > p.n3 - 1 - r) return;
    const long long g = ((long long)k * p.n2 + j) * p.pitch + i + (long long)s * p.fstride;
    const float *in[3] = {p.in1, p.in2, p.in3};
    // slab array index (layouts: x [n3][n2][2nb], y [n3][2nb][pitch], z [2nb][n2][pitch])
    long long id;
    float a, b;
    int c0, c1;  // the two input components with taps along this axis
    const float *A = REV_H ? p.a_half : p.a_int;
    const float *B = REV_H ? p.b_half : p.b_int;
    if (axis == 0) {
        id = ((long long)k * p.n2 + j) * nb2 + si + (long long)s * p.sxs;
        a = A[i];
        b = B[i];
        c0 = 1;
        c1 = 2;
    } else if (axis == 1) {
        id = ((long long)k * nb2 + si) * p.pitch + i + (long long)s * p.sys;
        a = A[p.n1 + j];
        b = B[p.n1 + j];
        c0 = 0;
        c1 = 2;
    } else {
        id = ((long long)si * p.n2 + j) * p.pitch + i + (long long)s * p.szs;
        a = A[p.n1 + p.n2 + k];
        b = B[p.n1 + p.n2 + k];
        c0 = 0;
        c1 = 1;
    }
    float *Q0 = p.Q[2 * axis], *Q1 = p.Q[2 * axis + 1];
    float *T0 = p.T[2 * axis], *T1 = p.T[2 * axis + 1];
    const float v0 = in[c0][g], v1 = in[c1][g];
    const float ps0 = b * Q0[id] + v0, ps1 = b * Q1[id] + v1;
    Q0[id] = ps0;
    Q1[id] = ps1;
    T0[id] = v0 + a * ps0;
    T1[id] = v1 + a * ps1;
}

// 2./3. transposed curl gathers, in the layout of the forward stencil
// kernel: a TX x (256/TX) tile of columns per 256-thread block marching a
// chunk of kz planes, x/y taps staged in LDS per plane (double-buffered,
// one barrier per plane, the next plane's loads issued right after it),
// z taps in a 2r-deep register queue.  Because the CPML reverse filter
// makes the tap value depend on the tap axis inside a slab, the staged
// copies are per (component, axis): the x taps of components 2 and 3 over
// the own rows with the x halo, the y taps of components 1 and 3 over the
// own columns with the y halo; every staged value is the filtered one (the
// slab array T inside the slab of its axis, the field elsewhere, zero off
// the update set on that axis).  CI (reverse of the H update only): dt/eps
// from the compact form, the table in LDS.
//
// As in step_kernel, memory bounds it on large grids and the vector unit on
// small ones, so a plane's accesses are a scalar base and a 32-bit column
// offset, the z queues turn by renaming, and elements off the update set are
// read where they lie (the fields are zero there, and so are the transposed
// tables' coefficients).  Only wavefronts that touch a slab read T.
// planes of loads in flight per thread: two at 8th order, as in step_kernel
template <int R, bool REV_H, bool CI, int TX, int PF = (R >= 4 ? 2 : 1)>
__global__ __launch_bounds__(kTileX * kTileY) void adj_tile(const AdjParams p) {
    constexpr int NT = kTileX * kTileY, TY = NT / TX;
    static_assert(TX * TY == NT && (TX & (TX - 1)) == 0, "tile of NT threads, power-of-two width");
    constexpr int L = 2 * R;
    static_assert(L % PF == 0, "the staged sets alternate within one turn of the z queues");
    constexpr int HL = REV_H ? R : R - 1;     // taps at q - HL .. q - HL + L - 1
    constexpr int W = TX + L - 1;
    constexpr int HR = TY + L - 1;
    constexpr int NX = (TY * W + NT - 1) / NT;        // x-type staging loads per thread
    constexpr int NY = (HR * TX + NT - 1) / NT;       // y-type staging loads per thread
    // x taps of components 3 and 2 [TY][W], y taps of 3 and 1 [HR][TX], each
    // with a spare word for threads without an element
    __shared__ float s3x[2][TY * W + 1], s2x[2][TY * W + 1];
    __shared__ float s3y[2][HR * TX + 1], s1y[2][HR * TX + 1];
    __shared__ float sCe[CI ? kCeTable : 1];
    static_assert(kCeTable <= NT, "one table entry per thread");
    // read only after the first barrier of the plane loop
    if (CI && (int)threadIdx.x < p.ncet) sCe[threadIdx.x] = p.cet[threadIdx.x];

    int t = xcd_tile(blockIdx.x, p.nstencil);
    const int s = uniform(tile_source(t, p.nsrc, p.nstencil, p.sorder));
    const int bxt = uniform(t % p.xt);
    t /= p.xt;
    const int byt = uniform(t % p.yt);
    const int bzt = uniform(t / p.yt);
    const int tid = threadIdx.x, tx = tid & (TX - 1), ty = tid / TX;
    const int i0 = bxt * TX, j0 = R + byt * TY;
    const int i = i0 + tx, j = j0 + ty;
    const int k0 = R + bzt * p.kz, k1 = min(k0 + p.kz, p.n3 - R);
    const bool valid = i >= R && i <= p.n1 - 1 - R && j <= p.n2 - 1 - R;
    const int jc = min(j, p.n2 - 1);
    const int nb = p.nb, nb2 = 2 * p.nb;
    const long long pb = 4ll * p.n2 * p.pitch;                 // bytes per plane
    const long long fo = (long long)s * p.fstride, cs = 4ll * p.nsrc * p.fstride;   // components of a field lie cs apart
    gchar *const A = (gchar *)(p.in1 + fo), *const O = (gchar *)(p.out1 + fo);
    // slab arrays of this source: x [n3][n2][2nb], y [n3][2nb][pitch], z [2nb][n2][pitch]
    gchar *const Tx2 = (gchar *)(p.T[0] + s * p.sxs), *const Tx3 = (gchar *)(p.T[1] + s * p.sxs);
    gchar *const Ty1 = (gchar *)(p.T[2] + s * p.sys), *const Ty3 = (gchar *)(p.T[3] + s * p.sys);
    gchar *const Tz1 = (gchar *)(p.T[4] + s * p.szs), *const Tz2 = (gchar *)(p.T[5] + s * p.szs);
    const long long xpb = 4ll * p.n2 * nb2, ypb = 4ll * nb2 * p.pitch;

    const int ic = valid ? i : R;
    float cx[L], cy[L];
#pragma unroll
    for (int m = 0; m < L; ++m) {
        cx[m] = p.tx[ic * L + m];
        cy[m] = p.ty[jc * L + m];
    }
    // slab index of update-set node q, or -1
    auto slab = [&](int q, int n) {
        return q < R || q > n - 1 - R ? -1 : q < nb ? q : q > n - 1 - nb ? q - (n - nb2) : -1;
    };
    auto at = [&](int gj, int gi) {
        return 4u * (unsigned)(min(max(gj, 0), p.n2 - 1) * p.pitch + min(max(gi, 0), p.pitch - 1));
    };
    // x-type element u: own row ly, column i0 - HL + lx; y-type: row j0 - HL +
    // ly, own column.  Byte offset in the field's plane, and in the slab
    // array's plane (~0u: not in a slab).
    unsigned xo[NX], xt[NX], yo[NY], yt[NY];
    bool xany[NX], yany[NY];
#pragma unroll
    for (int u = 0; u < NX; ++u) {
        const int e = tid + u * NT;
        const int ly = e / W, lx = e - ly * W;
        const int gj = min(j0 + ly, p.n2 - 1), gi = i0 - HL + lx;
        const int si = e < TY * W ? slab(gi, p.n1) : -1;
        xo[u] = e < TY * W ? at(gj, gi) : at(j0, i0);
        xt[u] = si >= 0 ? 4u * (unsigned)(gj * nb2 + si) : ~0u;
        xany[u] = __any(si >= 0);
    }
#pragma unroll
    for (int u = 0; u < NY; ++u) {
        const int e = tid + u * NT;
        const int gj = j0 - HL + e / TX;
        const int si = e < HR * TX ? slab(gj, p.n2) : -1;
        yo[u] = e < HR * TX ? at(gj, i) : at(j0, i0);
        yt[u] = si >= 0 ? 4u * (unsigned)(si * p.pitch + i) : ~0u;
        yany[u] = __any(si >= 0);
    }
    const int lx_ = tid + (NX - 1) * NT < TY * W ? tid + (NX - 1) * NT : TY * W;       // last elements' LDS index
    const int ly_ = tid + (NY - 1) * NT < HR * TX ? tid + (NY - 1) * NT : HR * TX;
    unsigned own = 4u * (unsigned)(jc * p.pitch + i);
    // z-filtered values of components 1 and 2 at plane kk of the own column
    auto zval = [&](int kk, float &a, float &b) {
        const int sk = slab(kk, p.n3);
        gchar *q = sk >= 0 ? Tz1 + sk * pb : A + kk * pb;
        gchar *r = sk >= 0 ? Tz2 + sk * pb : A + kk * pb + cs;
        keep_v(own);
        a = ldp<false>(keep_s(q), own);
        b = ldp<false>(keep_s(r), own);
    };
    // z queues: plane k - HL + m of step k at index (k - k0 + m) % L
    float q1[L], q2[L];
    q1[L - 1] = q2[L - 1] = 0.f;
#pragma unroll
    for (int m = 0; m < L - 1; ++m) zval(k0 - HL + m, q1[m], q2[m]);
    gchar *const En = (gchar *)(REV_H ? nullptr : p.E_next + fo), *const Ep = (gchar *)(REV_H ? nullptr : p.E_prev + fo);
    gchar *const G = (gchar *)(REV_H ? nullptr : p.grad32 + (long long)s * 3 * p.gstride);
    const long long gs = 4 * p.gstride;

    // staged registers of a plane in flight; PF sets, so that the loads of PF
    // planes are in flight while one is computed
    struct Stage {
        float f3x[NX], f2x[NX], f3y[NY], f1y[NY], e1n, e2n;
        float o1, o2, o3, w1, w2, w3;
        float g[3], xa[3], xn[3], xp[3];      // FP32 gradient sums, raw Et, E^{n+1}, E^n (reverse of the E update)
        unsigned wi;
    };
    auto issue = [&](Stage &S, int k) {
        const long long kb = k * pb;
        keep_v(own);
#pragma unroll
        for (int u = 0; u < NX; ++u) keep_v(xo[u]);
#pragma unroll
        for (int u = 0; u < NY; ++u) keep_v(yo[u]);
        gchar *a = keep_s(A + kb);
#pragma unroll
        for (int u = 0; u < NY; ++u) S.f1y[u] = ldp<false>(a, yo[u]);
        if (!REV_H) S.xa[0] = ldp<false>(a, own);
        a = keep_s(a + cs);
#pragma unroll
        for (int u = 0; u < NX; ++u) S.f2x[u] = ldp<false>(a, xo[u]);
        if (!REV_H) S.xa[1] = ldp<false>(a, own);
        a = keep_s(a + cs);
#pragma unroll
        for (int u = 0; u < NX; ++u) S.f3x[u] = ldp<false>(a, xo[u]);
#pragma unroll
        for (int u = 0; u < NY; ++u) S.f3y[u] = ldp<false>(a, yo[u]);
        if (!REV_H) S.xa[2] = ldp<false>(a, own);
#pragma unroll
        for (int u = 0; u < NX; ++u)
            if (xany[u] && xt[u] != ~0u) {
                unsigned o = xt[u];
                keep_v(o);
                S.f2x[u] = ldp<false>(keep_s(Tx2 + k * xpb), o);
                S.f3x[u] = ldp<false>(keep_s(Tx3 + k * xpb), o);
            }
#pragma unroll
        for (int u = 0; u < NY; ++u)
            if (yany[u] && yt[u] != ~0u) {
                unsigned o = yt[u];
                keep_v(o);
                S.f1y[u] = ldp<false>(keep_s(Ty1 + k * ypb), o);
                S.f3y[u] = ldp<false>(keep_s(Ty3 + k * ypb), o);
            }
        zval(k - HL + L - 1, S.e1n, S.e2n);
        keep_v(own);
        a = keep_s(O + kb);
        S.o1 = ldp<false>(a, own);
        a = keep_s(a + cs);
        S.o2 = ldp<false>(a, own);
        S.o3 = ldp<false>(keep_s(a + cs), own);
        if (REV_H && CI) {
            S.wi = *(const guint *)(keep_s((gchar *)p.cei + kb) + own);
        } else if (REV_H) {
            S.w1 = ldp<false>(keep_s((gchar *)p.ce1 + kb), own);
            S.w2 = ldp<false>(keep_s((gchar *)p.ce2 + kb), own);
            S.w3 = ldp<false>(keep_s((gchar *)p.ce3 + kb), own);
        } else {
            // E^{n+1} and E^n (their difference times raw Et is formed when
            // the plane is computed, after the loads landed)
            gchar *xn = keep_s(En + kb), *xp = keep_s(Ep + kb), *g = keep_s(G + kb);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                S.xn[c] = ldp<false>(xn, own);
                S.xp[c] = ldp<false>(xp, own);
                S.g[c] = ldp<false>(g, own);
                xn = keep_s(xn + cs);
                xp = keep_s(xp + cs);
                g = keep_s(g + gs);
            }
        }
    };
    auto step = [&](Stage &S, int k, auto turn) {
        constexpr int V = decltype(turn)::value, B = V & 1;
        q1[(V + L - 1) % L] = S.e1n;
        q2[(V + L - 1) % L] = S.e2n;
        const cfloat *czp = uniform_table(p.tz + k * L);
        float cz[L];
#pragma unroll
        for (int m = 0; m < L; ++m) cz[m] = czp[m];
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            s3x[B][u < NX - 1 ? tid + u * NT : lx_] = S.f3x[u];
            s2x[B][u < NX - 1 ? tid + u * NT : lx_] = S.f2x[u];
        }
#pragma unroll
        for (int u = 0; u < NY; ++u) {
            s3y[B][u < NY - 1 ? tid + u * NT : ly_] = S.f3y[u];
            s1y[B][u < NY - 1 ? tid + u * NT : ly_] = S.f1y[u];
        }
        const float u1 = S.o1, u2 = S.o2, u3 = S.o3;
        float g[3], v[3];                     // gradient sums; dt/eps or E^{n+1} - E^n
        float xa[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            g[c] = S.g[c];
            xa[c] = S.xa[c];
            v[c] = REV_H ? (c == 0 ? S.w1 : c == 1 ? S.w2 : S.w3) : S.xn[c] - S.xp[c];
        }
        const unsigned vi = S.wi;
        __syncthreads();
        if (k + PF < k1) issue(S, k + PF);
        if (CI) {
            v[0] = sCe[vi & 255u];
            v[1] = sCe[(vi >> 8) & 255u];
            v[2] = sCe[(vi >> 16) & 255u];
        }
        const float *y3 = s3y[B] + ty * TX + tx, *y1 = s1y[B] + ty * TX + tx;
        const float *x3 = s3x[B] + ty * W + tx, *x2 = s2x[B] + ty * W + tx;
        float d2a3 = 0.f, d2a1 = 0.f, d1a3 = 0.f, d1a2 = 0.f, d3a2 = 0.f, d3a1 = 0.f;
#pragma unroll
        for (int m = 0; m < L; ++m) {
            d2a3 += cy[m] * y3[m * TX];
            d2a1 += cy[m] * y1[m * TX];
            d1a3 += cx[m] * x3[m];
            d1a2 += cx[m] * x2[m];
            d3a2 += cz[m] * q2[(V + m) % L];
            d3a1 += cz[m] * q1[(V + m) % L];
        }
        if (valid) {
            const float c1 = d2a3 - d3a2, c2 = d3a1 - d1a3, c3 = d1a2 - d2a1;
            keep_v(own);
            gchar *o = keep_s(O + k * pb);
            if (REV_H) {
                stp<false>(o, own, u1 + v[0] * p.scale * c1);
                o = keep_s(o + cs);
                stp<false>(o, own, u2 + v[1] * p.scale * c2);
                stp<false>(keep_s(o + cs), own, u3 + v[2] * p.scale * c3);
            } else {
                gchar *q = keep_s(G + k * pb);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    stp<false>(q, own, __builtin_fmaf(xa[c], v[c], g[c]));
                    q = keep_s(q + gs);
                }
                stp<false>(o, own, u1 - p.scale * c1);
                o = keep_s(o + cs);
                stp<false>(o, own, u2 - p.scale * c2);
                stp<false>(keep_s(o + cs), own, u3 - p.scale * c3);
            }
        }
    };
    Stage S[PF] = {};
#pragma unroll
    for (int f = 0; f < PF; ++f)
        if (k0 + f < k1) issue(S[f], k0 + f);
    // one turn of the queues per pass
    auto turn = [&](auto self, int k, auto v) -> bool {
        constexpr int V = decltype(v)::value;
        if constexpr (V < L) {
            if (k >= k1) return true;
            step(S[V % PF], k, v);
            return self(self, k + 1, std::integral_constant<int, V + 1>{});
        } else {
            return false;
        }
    };
    for (int k = k0; !turn(turn, k, std::integral_constant<int, 0>{}); k += L) {}
}

// grad += grad32 / (dt/eps), grad32 = 0, over every cell of every source
__global__ __launch_bounds__(AT) void adj_flush(const AdjParams p) {
    const long long t = (long long)blockIdx.x * AT + threadIdx.x;
    const long long per_src = 3 * p.gstride;
    if (t >= per_src * p.nsrc) return;
    const long long u = t % per_src;
    const int c = (int)(u / p.gstride);
    const long long g = u - (long long)c * p.gstride;
    const float *ce = c == 0 ? p.ce1 : (c == 1 ? p.ce2 : p.ce3);
    const float v = p.grad32[t];
    if (v != 0.f) {
        p.grad[t] += (double)v / (double)ce[g];
        p.grad32[t] = 0.f;
    }
}

// out[((c nd2 + kk) nd1 + jj) nd0 + ii] = (accumulate ? out : 0) - sum over
// sources s and the padded cells (k, j, i) of the update set that fold onto
// input cell (ii, jj, kk) (the padding layers onto the edge cells) of
// grad[s][c][k][j][i], in a fixed order: one block per output row, each thread
// summing its padded column over the sources, k and j that fold onto the row
// (up to 15^2 of them at the edges, coalesced in x), then the ends of the row
// in x, whose columns alone pass through LDS, so that a row may have any length.  One thread per output cell did 15^3 uncoalesced sums in a row: 674
// us per gradient on 128 x 128 x 96 nodes.
__global__ __launch_bounds__(AT) void adj_fold(const double *grad, double *out, int nsrc, long long fstride,
                                               long long plane, int pitch, int n1, int n2, int n3, int r, int nbe,
                                               int nd0, int nd1, int nd2, int accumulate) {
    extern __shared__ double ends[];          // sums of the padded columns that fold onto the row's two ends
    int b = blockIdx.x;
    const int jj = b % nd1;
    b /= nd1;
    const int kk = b % nd2, c = b / nd2;
    const int j0 = jj == 0 ? r : jj + nbe, j1 = jj == nd1 - 1 ? n2 - 1 - r : jj + nbe;
    const int k0 = kk == 0 ? r : kk + nbe, k1 = kk == nd2 - 1 ? n3 - 1 - r : kk + nbe;
    // (padding thinner than r: the outer input cells are off the update set)
    const int nj = max(0, j1 - j0 + 1), rows = nj * max(0, k1 - k0 + 1);
    const int side = max(0, nbe - r + 1);     // columns r .. nbe fold onto the first cell, as many onto the last
    const int lo = min(r, nbe + 1);           // first column that is, or folds onto, an input cell
    double *o = out + (((long long)c * nd2 + kk) * nd1 + jj) * nd0;
    for (int s = 0; s < nsrc; ++s) {          // one source's fold after another, whatever the grouping
        const bool add = s > 0 || accumulate;
        for (int i = lo + threadIdx.x; i <= n1 - 1 - lo; i += AT) {
            const double *g = grad + ((long long)s * 3 + c) * fstride + i;
            double acc = 0.0;                 // (the sums are zero off the update set)
#pragma unroll 8
            for (int q = 0; q < rows; ++q) acc += g[(long long)(k0 + q / nj) * plane + (long long)(j0 + q % nj) * pitch];
            const int ii = i - nbe;
            if (ii <= 0) ends[i - r] = acc;
            else if (ii >= nd0 - 1) ends[side + ii - (nd0 - 1)] = acc;
            else o[ii] = (add ? o[ii] : 0.0) - acc;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            const int ii = threadIdx.x ? nd0 - 1 : 0;
            double acc = 0.0;
            for (int i = 0; i < side; ++i) acc += ends[threadIdx.x * side + i];
            o[ii] = (add ? o[ii] : 0.0) - acc;
        }
        __syncthreads();
    }
}

void launch_adj_fold(const double *grad, double *out, int nsrc, long long fstride, long long plane, int pitch,
                     int n1, int n2, int n3, int r, int nbe, int nd0, int nd1, int nd2, bool accumulate,
                     hipStream_t st) {
    const dim3 grid((unsigned)(3 * nd1 * nd2)), block(AT);
    hipLaunchKernelGGL(adj_fold, grid, block, 2 * std::max(0, nbe - r + 1) * sizeof(double), st, grad, out, nsrc, fstride, plane,
                       pitch, n1, n2, n3, r, nbe, nd0, nd1, nd2, accumulate ? 1 : 0);
}

void launch_adj_flush(const AdjParams &p, hipStream_t st) {
    const long long total = 3 * p.gstride * p.nsrc;
    const dim3 grid((unsigned)((total + AT - 1) / AT)), block(AT);
    hipLaunchKernelGGL(adj_flush, grid, block, 0, st, p);
}

void launch_adj_filter(bool rev_h, const AdjParams &p, bool filter, const InjectParams &q, int n, hipStream_t st) {
    const long long per_src = (long long)2 * p.nb * ((long long)p.n3 * p.n2 + (long long)p.n3 * p.n1 +
                                                      (long long)p.n2 * p.n1);
    const int nfilter = filter ? (int)((per_src * p.nsrc + AT - 1) / AT) : 0;
    const int ninject = n >= 0 ? (q.ncells + AT - 1) / AT : 0;
    if (nfilter + ninject == 0) return;
    const dim3 grid((unsigned)(nfilter + ninject)), block(AT);
    if (rev_h) hipLaunchKernelGGL(adj_filter<true>, grid, block, 0, st, p, nfilter, q, n);
    else hipLaunchKernelGGL(adj_filter<false>, grid, block, 0, st, p, nfilter, q, n);
}

template <bool REV_H, bool CI, int TX>
static void tiled(int r, const AdjParams &p, hipStream_t st) {
    const dim3 grid(p.nstencil), block(kTileX * kTileY);
    switch (r) {
    case 1: hipLaunchKernelGGL((adj_tile<1, REV_H, CI, TX>), grid, block, 0, st, p); break;
    case 2: hipLaunchKernelGGL((adj_tile<2, REV_H, CI, TX>), grid, block, 0, st, p); break;
    case 3: hipLaunchKernelGGL((adj_tile<3, REV_H, CI, TX>), grid, block, 0, st, p); break;
    default: hipLaunchKernelGGL((adj_tile<4, REV_H, CI, TX>), grid, block, 0, st, p); break;
    }
}

void launch_adj_tile(int r, bool rev_h, const AdjParams &p, hipStream_t st) {
    const bool w32 = p.tw == 32;
    if (rev_h && p.cei) {
        if (w32) tiled<true, true, 32>(r, p, st);
        else tiled<true, true, 64>(r, p, st);
    } else if (rev_h) {
        if (w32) tiled<true, false, 32>(r, p, st);
        else tiled<true, false, 64>(r, p, st);
    } else {
        if (w32) tiled<false, false, 32>(r, p, st);
        else tiled<false, false, 64>(r, p, st);
    }
}

}  // namespace emm
