// Time loops of small grids in one launch (see resident_kernel).
#include "emm_resident.h"

#include "emm_rec.h"

#include <type_traits>

namespace emm {

namespace {

typedef unsigned long long word;
typedef __attribute__((address_space(1))) char gchar;
typedef __attribute__((address_space(1))) word gword;
typedef __attribute__((address_space(1))) float gfloat;

// Words of the mailbox carry a value and the half step it belongs to, so a
// reader that finds the tag it waits for has the value too: one trip through
// memory, no flag and no fence.  Agent scope: past the L2 of the own XCD.
__device__ __forceinline__ void post(gchar *base, unsigned off, float v, unsigned tag) {
    __hip_atomic_store((gword *)(base + off), (word)tag << 32 | __float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ word peek(const gchar *base, unsigned off) {
    return __hip_atomic_load((const gword *)(base + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same value, but made anew in step n: addresses that do not change over
// the steps would otherwise be computed ahead of the time loop and held in
// registers, of which there are none to spare.
__device__ __forceinline__ gchar *fresh(gchar *q, int n) {
    asm("" : "+s"(q) : "s"(n));
    return q;
}
__device__ __forceinline__ const cfloat *fresh(const cfloat *q, int n) {
    asm("" : "+s"(q) : "s"(n));
    return q;
}
__device__ __forceinline__ unsigned fresh(unsigned v, int n) {
    asm("" : "+v"(v) : "s"(n));
    return v;
}
__device__ __forceinline__ int fresh_uniform(int v, int n) {
    asm("" : "+s"(v) : "s"(n));
    return v;
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

}  // namespace

// All time steps of a small grid in one cooperative launch.  A launch per
// half step costs 6-10 us there whatever it does (launch, prologue, three or
// four planes of dependent loads).  Here one block per compute unit keeps a
// tile of whole x rows on the chip for the whole run (own values, dt/eps and
// CPML memories in registers, the six components with their halos in LDS),
// and half steps are held together by the neighbours' edges alone: each tile
// posts the rows and planes its four neighbours read, tagged with the half
// step, and waits for theirs.  A tile can run at most one half step ahead of
// a neighbour, so one word per cell suffices: a tile overwrites its edge of
// field F only after it received the other field from that neighbour, who
// computed it after a block barrier behind its last read of F.
//
// Threads: `groups` groups of whole wavefronts, each holding all columns of
// the tile for P planes.  Component c of field f lies in LDS slot 3 f + c,
// [tz + 2r - 1][ty + 2r - 1][n1] with the halo that the half step reading
// field f needs; slots are a fixed distance apart, so one address register
// serves the two components with taps along an axis.  One plane per thread
// leaves 128 registers for 16 wavefronts; more planes run with 8 and 256.
//
// What bounds it: the mail (1300 clocks there and back, 2000-2400 at 5000
// words per tile) and the LDS reads of the taps.  us per step, half-step
// launches -> resident: 20^3 nodes r = 1 11.0 -> 3.6, r = 2 12.5 -> 5.3, r = 3
// 12.7 -> 7.7; 37 x 29 x 23 13.2 -> 7.9; 48^3 r = 1 16.7 -> 6.8, r = 2 16.7 ->
// 11.7.  At r = 4 the halos do not fit in LDS beside the tile.
template <int R, int P>
__global__ __launch_bounds__(resident_threads(P)) void resident_kernel(const StepParams pe, const StepParams ph,
                                                               const ResidentParams x) {
    constexpr int L = 2 * R, NW = resident_words(P);
    constexpr int HE = R - 1, HH = R;         // halo below of the tiles of E (read with D+) and H (D-)
    __shared__ float lds[6 * kResSlot];
    __shared__ float ztab[2][kResTall][L + 2];
    __shared__ int2 rowlist[2][kResRows];     // sampled rows: offset in the field's three tiles | length << 16, sample offset
    static_assert(3 * kResSlot <= 65536, "offsets in a field's tiles take 16 bits (rowlist, wto)");
    __shared__ int nrow[2], s_stuck;
    const int n1 = pe.n1, n2 = pe.n2, n3 = pe.n3, pitch = pe.pitch, nb = pe.nb, nb2 = 2 * pe.nb;
    const int plane = (int)pe.plane;
    const long long fs = pe.fstride;
    const int nx = n1 - L, ny = n2 - L, nz = n3 - L;
    const int bz = uniform(blockIdx.x / x.gy), by = uniform(blockIdx.x - bz * x.gy);
    const int y0 = uniform(R + ny * by / x.gy), ty = uniform(R + ny * (by + 1) / x.gy - y0);
    const int z0 = uniform(R + nz * bz / x.gz), tz = uniform(R + nz * (bz + 1) / x.gz - z0);
    const bool ylo = by > 0, yhi = by < x.gy - 1, zlo = bz > 0, zhi = bz < x.gz - 1;
    const int rs = n1, zs = (x.ty + L - 1) * n1;              // LDS row and plane strides
    const int tid = threadIdx.x, threads = blockDim.x, gthreads = threads / x.groups;
    const int grp = uniform(tid / gthreads), c0 = tid - grp * gthreads;
    const int p0 = grp * P;                                    // first plane of this group
    const bool col = c0 < nx * ty;
    const int yy = col ? c0 / nx : 0, i = R + (col ? c0 % nx : 0), j = y0 + yy;
    const unsigned cell = (unsigned)(j * pitch + i);
    const int here = p0 < tz ? min(P, tz - p0) : 0;            // planes of this group in this tile

    for (int e = tid; e < 6 * kResSlot; e += threads) lds[e] = 0.f;
    if (tid < 2) nrow[tid] = 0;
    if (tid == 0) s_stuck = 0;
    __syncthreads();

    // ---- state of the columns
    float F[2][3][P], ce[3][P], M[2][3][2][P];                 // E and H, dt/eps, CPML memories
    const bool xs = col && (i < nb || i > n1 - 1 - nb), ys = col && (j < nb || j > n2 - 1 - nb);
    int src = x.src;
    unsigned cellv = cell, xcol = (unsigned)(j * nb2 + (i < nb ? i : i - (n1 - nb2))),
             ycol = (unsigned)((j < nb ? j : j - (n2 - nb2)) * pitch + i);
    auto field_at = [&](int h, int c, int k) -> float * {
        const StepParams &q = h ? ph : pe;
        float *f = h ? (c == 0 ? q.H1 : c == 1 ? q.H2 : q.H3) : (c == 0 ? q.E1 : c == 1 ? q.E2 : q.E3);
        return f + (src * fs + (long long)k * plane) + cellv;
    };
    auto mem_at = [&](int h, int a, int d, int k) -> float * {
        const StepParams &q = h ? ph : pe;
        if (a == 0) return (d ? q.psx1 : q.psx0) + (src * q.psxs + (long long)k * n2 * nb2) + xcol;
        if (a == 1) return (d ? q.psy1 : q.psy0) + (src * q.psys + (long long)k * nb2 * pitch) + ycol;
        const int kz = k < nb ? k : k - (n3 - nb2);
        return (d ? q.psz1 : q.psz0) + (src * q.pszs + (long long)kz * plane) + cellv;
    };
    auto zslab = [&](int k) { return k < nb || k > n3 - 1 - nb; };
    auto slab = [&](int a, int k) { return a == 0 ? xs : a == 1 ? ys : zslab(k); };
    // LDS offset of the column's cell of plane p, tiles of E (h = 0) and H (h = 1)
    auto at = [&](int h, int p) { return (unsigned)((p + (h ? HH : HE)) * zs + (yy + (h ? HH : HE)) * rs + i); };
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const bool live = col && p < here;
        const int k = z0 + p0 + p;
        const unsigned g = (unsigned)(k * plane) + cell;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            F[0][c][p] = live ? *field_at(0, c, k) : 0.f;
            F[1][c][p] = live ? *field_at(1, c, k) : 0.f;
            ce[c][p] = live ? (c == 0 ? pe.ce1 : c == 1 ? pe.ce2 : pe.ce3)[g] : 0.f;
            if (live) {
                lds[c * kResSlot + at(0, p0 + p)] = F[0][c][p];
                lds[(3 + c) * kResSlot + at(1, p0 + p)] = F[1][c][p];
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int d = 0; d < 2; ++d) M[h][a][d][p] = live && slab(a, k) ? *mem_at(h, a, d, k) : 0.f;
    }
    float cx[2][L], cy[2][L];                                  // D- (E step), D+ (H step)
    float ax[2] = {}, bx[2] = {}, ay[2] = {}, by_[2] = {};
#pragma unroll
    for (int m = 0; m < L; ++m) {
        cx[0][m] = pe.cmx[i * L + m];
        cx[1][m] = ph.cpx[i * L + m];
        cy[0][m] = pe.cmy[j * L + m];
        cy[1][m] = ph.cpy[j * L + m];
    }
    if (xs) {
        ax[0] = pe.axi[i];
        bx[0] = pe.bxi[i];
        ax[1] = ph.axh[i];
        bx[1] = ph.bxh[i];
    }
    if (ys) {
        ay[0] = pe.ayi[j];
        by_[0] = pe.byi[j];
        ay[1] = ph.ayh[j];
        by_[1] = ph.byh[j];
    }
    // dipole of this source on the column
    const int scomp = pe.src_info[4 * x.src], sbx = pe.src_info[4 * x.src + 1], sby = pe.src_info[4 * x.src + 2],
              sbz = pe.src_info[4 * x.src + 3];
    const bool scol = col && j >= sby && j < sby + L && i >= sbx && i < sbx + L;
    const float *sq = pe.src_q + (long long)x.src * L * L * L + (scol ? (j - sby) * L + (i - sbx) : 0);

    const bool wsrc = __any(scol);
    float ch = ph.ch;
    asm("" : "+v"(ch));                       // in a register, not read again in every step
    // z rows of the tables and the z slabs' a, b (zero elsewhere), E and H step
    for (int q = tid; q < 2 * tz * (L + 2); q += threads) {
        const int h = q / (tz * (L + 2)), pl = q / (L + 2) % tz, m = q % (L + 2), k = z0 + pl;
        ztab[h][pl][m] = m < L ? (h ? ph.cpz : pe.cmz)[k * L + m]
                       : zslab(k) ? (m == L ? (h ? ph.azh : pe.azi) : (h ? ph.bzh : pe.bzi))[k] : 0.f;
    }

    // ---- the words this thread receives: word w of the tile's 2 (2r - 1)
    // (ty + tz) nx, of which the first 2 (2r - 1) ty nx are z halo (components
    // 1, 2), the others y halo (1, 3).  Byte offset of the word in the mail
    // of the field, LDS offset in its slots; ~0u: none (or off the grid).
    unsigned wfrom[2][NW];
    unsigned short wto[2][NW];
#pragma unroll
    for (int h = 0; h < 2; ++h)                                // h: field received (0: E, 1: H)
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int HL = h ? HH : HE;
            const int w = tid + q * threads;
            const int unit = w / nx, xi = R + w - unit * nx, nzu = 2 * (L - 1) * ty;
            int c, m, yl, zl;                                  // component, halo index, LDS row and plane
            bool in;
            if (unit < nzu) {
                m = unit % (L - 1);
                yl = HL + unit / (L - 1) % ty;
                c = unit / ((L - 1) * ty);
                zl = m < HL ? m : m + tz;
                in = m < HL ? zlo : zhi;
            } else {
                const int v = unit - nzu;
                m = v % (L - 1);
                zl = HL + v / (L - 1) % tz;
                c = 2 * (v / ((L - 1) * tz));
                yl = m < HL ? m : m + ty;
                in = (m < HL ? ylo : yhi) && v < 2 * (L - 1) * tz;
            }
            const unsigned word_at = (unsigned)((z0 + zl - HL) * plane + (y0 + yl - HL) * pitch + xi);
            wfrom[h][q] = in ? 8u * (c * (unsigned)fs + word_at) : ~0u;
            wto[h][q] = (unsigned short)(c * kResSlot + zl * zs + yl * rs + xi);
        }
    gchar *const mail = (gchar *)x.mail;

    // ---- rows of the tile that receivers read
    for (int h = 0; h < 2; ++h)                                // h = 0: rows of H, read in the E step
        for (int q = tid; q < x.nrows[h]; q += threads) {
            const ResidentRow w = x.rows[h][q];
            if (w.y < y0 || w.y >= y0 + ty || w.z < z0 || w.z >= z0 + tz) continue;
            const int slot = atomicAdd(&nrow[h], 1), HL = h ? HE : HH;
            if (slot < kResRows)
                rowlist[h][slot] = make_int2((w.comp * kResSlot + (w.z - z0 + HL) * zs + (w.y - y0 + HL) * rs + w.x0) |
                                                 w.len << 16, w.off);
            else s_stuck = 1;
        }

    // edges of field h (0: E, 1: H) that the neighbours read next
    auto edges = [&](int h, int p, unsigned tag, int n) {
        const int CL = h ? HH : HE, CH = L - 1 - CL;
        const int pl = p0 + p;
        const bool ypub = (yy < CH && ylo) || (yy >= ty - CL && yhi);
        const bool zpub = (pl < CH && zlo) || (pl >= tz - CL && zhi);
        const unsigned off = 8u * fresh(cell, n);
        gchar *o = fresh(mail + 8 * ((h ? 3 * fs : 0) + (long long)(z0 + pl) * plane), n);
        if (ypub || zpub) post(o, off, F[h][0][p], tag);
        o = fresh(o + 8 * fs, n);
        if (zpub) post(o, off, F[h][1][p], tag);
        o = fresh(o + 8 * fs, n);
        if (ypub) post(o, off, F[h][2][p], tag);
    };

    // One half step.  HS = 0: E from H; 1: H from E.  tag: that of the field
    // read; the updated field gets the next.
    auto half = [&](auto hs, int n, unsigned tag) -> bool {
        constexpr int HS = decltype(hs)::value, A = 1 - HS;    // A: the field read
        constexpr int HL = A ? HH : HE;
        float *const sA = lds + 3 * A * kResSlot, *const sU = lds + 3 * HS * kResSlot;
        // ---- receive the halo
        {
            const unsigned long long t0 = wall_clock64();
            word got[NW];
            const word blank = (word)tag << 32;
            for (;;) {
                bool miss = false;
                gchar *from = fresh(mail + (A ? 24 * fs : 0), n);
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    got[q] = blank;
                    if (wfrom[A][q] != ~0u) got[q] = peek(from, fresh(wfrom[A][q], n));
                }
#pragma unroll
                for (int q = 0; q < NW; ++q) miss |= (unsigned)(got[q] >> 32) != tag;
                if (!__any(miss)) break;
                if (wall_clock64() - t0 > x.patience) {
                    s_stuck = 1;
                    break;
                }
            }
#pragma unroll
            for (int q = 0; q < NW; ++q)
                if (wfrom[A][q] != ~0u) sA[wto[A][q]] = __uint_as_float((unsigned)got[q]);
        }
        __syncthreads();
        // (a wave behind may see the flag of one that gave up a half step ahead
        // and leave before it: a barrier waits for the surviving waves only,
        // and wave 0 sees the flag at the latest at the barrier that follows)
        if (s_stuck) return false;

        // ---- compute, post the tile's edges (without branches up to there:
        // threads without a column and planes off the tile compute a copy of
        // another's, lanes off the slabs filter with zeros)
        const float sn = HS ? 0.f : pe.wavelet[n];
        const int rn = fresh_uniform(rs, n), zn = fresh_uniform(zs, n);
        const unsigned o0 = fresh((unsigned)(HL * zs + (yy + HL) * rs + i) + p0 * zn, n);
        // the column of components 1 and 2, halo planes and all (planes past
        // the tile's last only feed what is not stored; resident_reach keeps
        // their taps inside the array)
        float g1[P + L - 1], g2[P + L - 1];
#pragma unroll
        for (int q = 0; q < P + L - 1; ++q) {
            const float *o = sA + o0 + (q - HL) * zn;
            g1[q] = o[0];
            g2[q] = o[kResSlot];
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma clang fp contract(off)
            const int pl = min(p0 + p, tz - 1), k = z0 + pl;
            const float *o = sA + o0 + p * zn, *zt = ztab[HS][pl];
            float d2a3 = 0.f, d2a1 = 0.f, d1a3 = 0.f, d1a2 = 0.f, d3a2 = 0.f, d3a1 = 0.f;
#pragma unroll
            for (int m = 0; m < L; ++m) {
                const float *oy = o + (m - HL) * rn, *ox = o + (m - HL);
                d2a3 = __builtin_fmaf(cy[HS][m], oy[2 * kResSlot], d2a3);
                d2a1 = __builtin_fmaf(cy[HS][m], m == HL ? g1[p + HL] : oy[0], d2a1);
                d1a3 = __builtin_fmaf(cx[HS][m], ox[2 * kResSlot], d1a3);
                d1a2 = __builtin_fmaf(cx[HS][m], m == HL ? g2[p + HL] : ox[kResSlot], d1a2);
                d3a2 = __builtin_fmaf(zt[m], g2[p + m], d3a2);
                d3a1 = __builtin_fmaf(zt[m], g1[p + m], d3a1);
            }
            auto filter = [&](float &mv, float a, float b, float &d) {
                mv = __builtin_fmaf(b, mv, a * d);
                d += mv;
            };
            filter(M[HS][0][0][p], ax[HS], bx[HS], d1a3);
            filter(M[HS][0][1][p], ax[HS], bx[HS], d1a2);
            filter(M[HS][1][0][p], ay[HS], by_[HS], d2a3);
            filter(M[HS][1][1][p], ay[HS], by_[HS], d2a1);
            filter(M[HS][2][0][p], zt[L], zt[L + 1], d3a2);
            filter(M[HS][2][1][p], zt[L], zt[L + 1], d3a1);
            float c1 = d2a3 - d3a2, c2 = d3a1 - d1a3, c3 = d1a2 - d2a1;
            if (!HS && wsrc && k >= sbz && k < sbz + L && scol) {
                const float jv = sn * sq[(k - sbz) * L * L];
                if (scomp == 0) c1 -= jv;
                else if (scomp == 1) c2 -= jv;
                else c3 -= jv;
            }
            F[HS][0][p] = __builtin_fmaf(HS ? -ch : ce[0][p], c1, F[HS][0][p]);
            F[HS][1][p] = __builtin_fmaf(HS ? -ch : ce[1][p], c2, F[HS][1][p]);
            F[HS][2][p] = __builtin_fmaf(HS ? -ch : ce[2][p], c3, F[HS][2][p]);
        }
        if (col) {
            // the updated field's halo differs by one row and plane from the other's
            float *u = sU + o0 + ((HS ? HH : HE) - HL) * (zn + rn);
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (p < here) {
                    edges(HS, p, tag + 1, n);
                    u[p * zn] = F[HS][0][p];
                    u[p * zn + kResSlot] = F[HS][1][p];
                    u[p * zn + 2 * kResSlot] = F[HS][2][p];
                }
        }
        if (!HS && x.snap && col) {
            gchar *o = (gchar *)(x.snap + (n - x.n0) * x.snap_stride + x.src * fs + (long long)(z0 + p0) * plane);
            const unsigned off = 4u * fresh(cell, n);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                gchar *q = fresh(o, n);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    if (p < here) *(gfloat *)(q + off) = F[0][c][p];
                    q = fresh(q + 4ll * plane, n);
                }
                o += 4 * pe.nsrc * fs;
            }
        }
        // ---- samples of the field read, while the mail travels
        const int cnt = nrow[HS];
        float *smp = x.samples + (long long)(n - x.nbase) * x.per_step;
        for (int q = uniform(tid >> 6); q < cnt; q += threads >> 6) {
            const int2 d = rowlist[HS][q];
            const int len = d.x >> 16 & 0xffff;
            for (int e = tid & 63; e < len; e += 64) smp[d.y + e] = sA[(d.x & 0xffff) + e];
        }
        return true;
    };

    unsigned tag = x.tag;
    if (col)
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (p < here) edges(1, p, tag, x.n0);
    bool fine = true;
    for (int n = x.n0; fine && n < x.n1; ++n, tag += 2)
        fine = half(std::integral_constant<int, 0>{}, n, tag) && half(std::integral_constant<int, 1>{}, n, tag + 1);
    if (!fine) {
        if (tid == 0) *x.stuck = 1;
        return;
    }
    src = fresh_uniform(src, x.n1);
    const int z0n = fresh_uniform(z0, x.n1);
    cellv = fresh(cellv, x.n1);
    xcol = fresh(xcol, x.n1);
    ycol = fresh(ycol, x.n1);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int k = z0n + p0 + p;
        if (!col || p >= here) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            *field_at(0, c, k) = F[0][c][p];
            *field_at(1, c, k) = F[1][c][p];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int d = 0; d < 2; ++d)
                    if (slab(a, k)) *mem_at(h, a, d, k) = M[h][a][d][p];
    }
}

template <int R, int P>
static hipError_t resident(const ResidentPlan &plan, StepParams pe, StepParams ph, ResidentParams x, hipStream_t s) {
    void *args[] = {&pe, &ph, &x};
    return hipLaunchCooperativeKernel((const void *)resident_kernel<R, P>, dim3(plan.gy * plan.gz), dim3(plan.threads),
                                      args, 0, s);
}

template <int R>
static hipError_t resident(const ResidentPlan &plan, const StepParams &pe, const StepParams &ph,
                           const ResidentParams &x, hipStream_t s) {
    switch (plan.planes) {
    case 1: return resident<R, 1>(plan, pe, ph, x, s);
    case 2: return resident<R, 2>(plan, pe, ph, x, s);
    case 3: return resident<R, 3>(plan, pe, ph, x, s);
    case 4: return resident<R, 4>(plan, pe, ph, x, s);
    default: return resident<R, 5>(plan, pe, ph, x, s);
    }
}

hipError_t launch_resident(int r, const ResidentPlan &plan, const StepParams &pe, const StepParams &ph,
                           const ResidentParams &x, hipStream_t s) {
    switch (r) {
    case 1: return resident<1>(plan, pe, ph, x, s);
    case 2: return resident<2>(plan, pe, ph, x, s);
    default: return resident<3>(plan, pe, ph, x, s);
    }
}

// u of every (step, item): one wavefront each
template <int R>
__global__ __launch_bounds__(256) void resident_sum(const StepParams pe, const StepParams ph, const ResidentParams x,
                                                    double *u) {
    constexpr int L = 2 * R;
    const int nit = x.nitems[0] + x.nitems[1];
    const long long q = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q >= (long long)(x.n1 - x.n0) * nit) return;
    const int n = x.n0 + (int)(q / nit), it = (int)(q % nit);
    const int h = it >= x.nitems[0], mine = h ? it - x.nitems[0] : it;
    const StepParams &P = h ? ph : pe;
    const float *s = x.samples + (long long)(n - x.nbase) * x.per_step;
    const int *row = x.item_rows[h] + mine * (L * L);
    const double v = rec_sum<R>(P.item_w + 3 * L * (mine * P.nsrc + x.src), threadIdx.x & 63,
                                [&](int, int a, int b, int c) {
                                    const int at = row[c * L + b];
                                    return at < 0 ? 0.f : s[at + a];
                                });
    if ((threadIdx.x & 63) == 0) u[(long long)(n - x.nbase) * nit + it] = v;
}

// accumulators: one thread per (item, frequency), the steps in order
template <typename Acc>
__global__ __launch_bounds__(64) void resident_acc(const StepParams pe, const StepParams ph, const ResidentParams x,
                                                   const double *u) {
    const int nit = x.nitems[0] + x.nitems[1], nf = pe.nf;
    const int q = blockIdx.x * 64 + threadIdx.x;
    if (q >= nit * nf) return;
    const int it = q / nf, f = q % nf;
    const int h = it >= x.nitems[0], mine = h ? it - x.nitems[0] : it;
    const StepParams &P = h ? ph : pe;
    const long long k = (long long)P.item_info[6 * (mine * P.nsrc + x.src) + 5] * nf + f;
    Acc *acc = std::is_same<Acc, float4>::value ? (Acc *)P.acck : (Acc *)P.acc;
    Acc a = acc[k];
#pragma unroll 8
    for (int n = x.n0; n < x.n1; ++n) rec_add(a, u[(long long)(n - x.nbase) * nit + it], P.phase[(long long)n * nf + f]);
    acc[k] = a;
}

void launch_resident_dft(int r, const StepParams &pe, const StepParams &ph, const ResidentParams &x, double *u,
                         hipStream_t s) {
    const int nit = x.nitems[0] + x.nitems[1];
    const long long waves = (long long)(x.n1 - x.n0) * nit;
    if (waves == 0) return;
    const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
    switch (r) {
    case 1: hipLaunchKernelGGL(resident_sum<1>, grid, block, 0, s, pe, ph, x, u); break;
    case 2: hipLaunchKernelGGL(resident_sum<2>, grid, block, 0, s, pe, ph, x, u); break;
    default: hipLaunchKernelGGL(resident_sum<3>, grid, block, 0, s, pe, ph, x, u); break;
    }
    const dim3 ga((nit * pe.nf + 63) / 64), ba(64);
    if (pe.dft_mode) hipLaunchKernelGGL(resident_acc<float4>, ga, ba, 0, s, pe, ph, x, u);
    else hipLaunchKernelGGL(resident_acc<double2>, ga, ba, 0, s, pe, ph, x, u);
}

}  // namespace emm
