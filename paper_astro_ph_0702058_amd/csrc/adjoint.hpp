// adjoint.hpp -- gfx950 device code for differentiating shared-step Hermite runs.
//
// One shared step of the Sec. 2 scheme with fixed dt, written out as a map of the state
// (x, v, a, k) and the new force (a1, k1) = F(x_p, v_p, m) at the predicted state:
//   x_p = x + dt v + dt^2/2 a + dt^3/6 k,         v_p = v + dt a + dt^2/2 k,
//   x'  = x + dt v + 7/20 dt^2 a + 3/20 dt^2 a1 + 1/20 dt^3 k - 1/30 dt^3 k1,
//   v'  = v + dt/2 (a + a1) + dt^2/12 (k - k1),    a' = a1,  k' = k1
// (the corrector's a2 dt^4/24 + a3 dt^5/120 and a2 dt^3/6 + a3 dt^4/24 expanded).  Its
// vector-Jacobian product is the transposed linear part plus the VJP of F, whose pair form is
//   phi(d, u; A, B) = A.d s^-3/2 + B.u s^-3/2 - 3 (d.u)(B.d) s^-5/2
// (A, B: adjoints of the acceleration and jerk of i; d = x_j - x_i, u = v_j - v_i), with
//   dphi/dd = A s^-3/2 - 3 s^-5/2 [(A.d + B.u) d + (B.d) u + (d.u) B] + 15 s^-7/2 (d.u)(B.d) d
//   dphi/du = B s^-3/2 - 3 s^-5/2 (B.d) d,      dphi/dm_j = phi / m_j.
// Every particle p gathers, over all q != p, its i-side terms (A_p, B_p against q) and its
// j-side terms (A_q, B_q of q against p).
#pragma once

#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace nbody {

// Predictor of every particle over the shared step dt, into the j-particle stream.
template <int MODE>
__global__ void __launch_bounds__(WG) shared_predict(StateView s, JStreamView js, double dt) {
    const int32_t n = s.n;
    for (int32_t i = blockIdx.x * WG + threadIdx.x; i < n; i += gridDim.x * WG) {
        double xp[3], vp[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            predict_one(dt, s.x[c * (int64_t)n + i], s.v[c * (int64_t)n + i],
                        s.a[c * (int64_t)n + i], s.k[c * (int64_t)n + i], xp[c], vp[c]);
        const double m = s.m[i];
        if (MODE == 0) {
            js.px[i] = xp[0]; js.py[i] = xp[1]; js.pz[i] = xp[2];
            js.vm[i] = make_float4((float)vp[0], (float)vp[1], (float)vp[2], (float)m);
        } else {
            js.px[i] = xp[0]; js.py[i] = xp[1]; js.pz[i] = xp[2]; js.pm[i] = m;
            js.vx[i] = vp[0]; js.vy[i] = vp[1]; js.vz[i] = vp[2];
        }
    }
}

// Corrector of every particle over the shared step dt (advances each time by dt_ticks).
__global__ void __launch_bounds__(WG) shared_correct(StateRW s, const double *acc,
                                                     const double *jerk, const double *pot,
                                                     double dt, int64_t dt_ticks,
                                                     int32_t *flag) {
    const int32_t n = s.n;
    for (int32_t i = blockIdx.x * WG + threadIdx.x; i < n; i += gridDim.x * WG) {
        double a1[3], k1[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a1[c] = acc[c * (int64_t)n + i];
            k1[c] = jerk[c * (int64_t)n + i];
        }
        if (!correct_particle(s, i, dt, a1, k1, pot[i], s.tick[i] + dt_ticks, nullptr)) *flag = 1;
    }
}

// Step VJP, first part: adjoints of the new force from those of the step's outputs.
//   a1_bar = 3/20 dt^2 x'_bar + dt/2 v'_bar + a'_bar,  k1_bar = -1/30 dt^3 x'_bar - dt^2/12 v'_bar + k'_bar
__global__ void __launch_bounds__(WG) vjp_pre(int32_t n, double dt, const double *xb,
                                              const double *vb, const double *ab,
                                              const double *kb, double *a1b, double *k1b) {
    const double dt2 = dt * dt, dt3 = dt2 * dt;
    for (int64_t e = blockIdx.x * (int64_t)WG + threadIdx.x; e < 3 * (int64_t)n;
         e += (int64_t)gridDim.x * WG) {
        a1b[e] = (3.0 / 20.0) * dt2 * xb[e] + 0.5 * dt * vb[e] + ab[e];
        k1b[e] = -(1.0 / 30.0) * dt3 * xb[e] - (1.0 / 12.0) * dt2 * vb[e] + kb[e];
    }
}

// Step VJP, last part: adjoints of the step's inputs, in place, from those of its outputs and
// of the predicted state (xpb, vpb: the force VJP).
__global__ void __launch_bounds__(WG) vjp_post(int32_t n, double dt, double *xb, double *vb,
                                               double *ab, double *kb, const double *xpb,
                                               const double *vpb) {
    const double dt2 = dt * dt, dt3 = dt2 * dt;
    for (int64_t e = blockIdx.x * (int64_t)WG + threadIdx.x; e < 3 * (int64_t)n;
         e += (int64_t)gridDim.x * WG) {
        const double X = xb[e], V = vb[e], XP = xpb[e], VP = vpb[e];
        xb[e] = X + XP;
        vb[e] = dt * X + V + dt * XP + VP;
        ab[e] = (7.0 / 20.0) * dt2 * X + 0.5 * dt * V + 0.5 * dt2 * XP + dt * VP;
        kb[e] = (1.0 / 20.0) * dt3 * X + (1.0 / 12.0) * dt2 * V + (1.0 / 6.0) * dt3 * XP +
                0.5 * dt2 * VP;
    }
}

template <class T> __device__ __forceinline__ T fma_t(T a, T b, T c);
template <> __device__ __forceinline__ float fma_t<float>(float a, float b, float c) {
    return __builtin_fmaf(a, b, c);
}
template <> __device__ __forceinline__ double fma_t<double>(double a, double b, double c) {
    return __builtin_fma(a, b, c);
}

// Pair terms of the force VJP for particle p against q, arithmetic type T.  d = x_q - x_p,
// u = v_q - v_p; (A, B) adjoints of p, (Aq, Bq) adjoints of q; rinv = s^-1/2 or 0 (self).
// With r3 = rinv^3, r5, r7 and du = d.u, the derivative of m_q (A.a + B.k) with respect to d
// is m_q [A r3 + c1 d + c2 u + c3 B] and with respect to u is m_q [B r3 + c2 d], where
// c1 = -3 r5 (A.d + B.u) + 15 r7 du B.d, c2 = -3 r5 B.d, c3 = -3 r5 du (even in (d, u)).
// p gains the i-side term with -m_q and its own (A, B), and the j-side term with +m_p and
// q's (Aq, Bq); both are added at once, the shared factors formed once:
//   gx += r3 (m_p Aq - m_q A) + (m_p c1q - m_q c1) d + (m_p c2q - m_q c2) u + c3 (m_p Bq - m_q B)
//   gu += r3 (m_p Bq - m_q B) + (m_p c2q - m_q c2) d
// and gm gains phi at (-d, -u) with q's adjoints: -(Aq.d + Bq.u) r3 - c3 Bq.d.
// p's adjoints come in negated (nA = -A, nB = -B) and the mass sum is kept negated (ngm = -gm):
// round-to-nearest is odd-symmetric, so every value is exactly the one the signs above give,
// and each product with a negated operand is a plain two-operand multiply or FMA rather than
// one carrying a negation modifier (which takes the slower three-operand encoding).
template <class T>
struct VjpTerms {
    T r3, C1, C2, c3, d[3], u[3], Ab[3], Bb[3], abq, bdq;  // abq = Aq.d + Bq.u, bdq = Bq.d
};
template <class T>
__device__ __forceinline__ VjpTerms<T> vjp_terms(T dx, T dy, T dz, T ux, T uy, T uz, T rinv, T mp,
                                                 T mq, const T nA[3], const T nB[3],
                                                 const T Aq[3], const T Bq[3]) {
    const T r2 = rinv * rinv, r3 = rinv * r2, r5 = r3 * r2, r7 = r5 * r2;
    const T du = fma_t(dz, uz, fma_t(dy, uy, dx * ux));
    const T m3r5 = T(-3) * r5;
    const T c3 = m3r5 * du;
    const T f15 = (T(15) * r7) * du;
    const T nAd = fma_t(nA[2], dz, fma_t(nA[1], dy, nA[0] * dx));  // -A.d
    const T nBd = fma_t(nB[2], dz, fma_t(nB[1], dy, nB[0] * dx));  // -B.d
    const T nBu = fma_t(nB[2], uz, fma_t(nB[1], uy, nB[0] * ux));  // -B.u
    const T nc1 = fma_t(f15, nBd, m3r5 * (nAd + nBu));             // -c1
    const T nc2 = m3r5 * nBd;                                       // -c2
    const T Adq = fma_t(Aq[2], dz, fma_t(Aq[1], dy, Aq[0] * dx));
    const T Bdq = fma_t(Bq[2], dz, fma_t(Bq[1], dy, Bq[0] * dx));
    const T Buq = fma_t(Bq[2], uz, fma_t(Bq[1], uy, Bq[0] * ux));
    const T abq = Adq + Buq;
    const T c1q = fma_t(f15, Bdq, m3r5 * abq);
    const T c2q = m3r5 * Bdq;
    VjpTerms<T> o{r3, fma_t(mp, c1q, mq * nc1), fma_t(mp, c2q, mq * nc2), c3,
                  {dx, dy, dz}, {ux, uy, uz}, {}, {}, abq, Bdq};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        o.Ab[k] = fma_t(mp, Aq[k], mq * nA[k]);
        o.Bb[k] = fma_t(mp, Bq[k], mq * nB[k]);
    }
    return o;
}

template <class T>
struct VjpSum {
    T gx[3] = {0, 0, 0}, gu[3] = {0, 0, 0}, ngm = 0;
    __device__ __forceinline__ void add(const VjpTerms<T> &o) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            gx[k] = fma_t(o.r3, o.Ab[k], fma_t(o.C1, o.d[k], fma_t(o.C2, o.u[k], fma_t(o.c3, o.Bb[k], gx[k]))));
            gu[k] = fma_t(o.r3, o.Bb[k], fma_t(o.C2, o.d[k], gu[k]));
        }
        ngm = fma_t(o.abq, o.r3, fma_t(o.c3, o.bdq, ngm));
    }
};

// Adds the terms of the four lanes of a quad to every lane's g, in lane order: each addition is
// the one VjpSum::add makes, with the other lane's values as DPP operands.  The four lanes hold
// the same g.  (A DPP operand is read two wait states after it was written: the s_nop.)
#define NB_QUAD(n) " quad_perm:[" n "," n "," n "," n "] row_mask:0xf bank_mask:0xf\n"
#define NB_F3(a, b, c, x, y, z, m, n)                                                         \
    "v_fmac_f32_dpp %" a ", %" x ", %" m NB_QUAD(n) "v_fmac_f32_dpp %" b ", %" y ", %" m      \
    NB_QUAD(n) "v_fmac_f32_dpp %" c ", %" z ", %" m NB_QUAD(n)
#define NB_VJP_GX(n)                                                                          \
    "v_mov_b32_dpp %3, %22" NB_QUAD(n) "v_mov_b32_dpp %4, %21" NB_QUAD(n)                     \
    "v_mov_b32_dpp %5, %20" NB_QUAD(n) "v_mov_b32_dpp %6, %19" NB_QUAD(n)                     \
    NB_F3("0", "1", "2", "16", "17", "18", "3", n) NB_F3("0", "1", "2", "10", "11", "12", "4", n) \
    NB_F3("0", "1", "2", "7", "8", "9", "5", n) NB_F3("0", "1", "2", "13", "14", "15", "6", n)
#define NB_VJP_GU(n)                                                                          \
    "v_mov_b32_dpp %4, %17" NB_QUAD(n) "v_mov_b32_dpp %5, %16" NB_QUAD(n)                     \
    "v_mov_b32_dpp %6, %15" NB_QUAD(n)                                                        \
    NB_F3("0", "1", "2", "7", "8", "9", "5", n) "v_fmac_f32_dpp %3, %14, %4" NB_QUAD(n)       \
    NB_F3("0", "1", "2", "10", "11", "12", "6", n) "v_fmac_f32_dpp %3, %13, %6" NB_QUAD(n)
__device__ __forceinline__ void vjp_add_quad(VjpSum<float> &g, const VjpTerms<float> &o) {
    float m0, m1, m2, m3;
    asm("s_nop 1\n" NB_VJP_GX("0") NB_VJP_GX("1") NB_VJP_GX("2") NB_VJP_GX("3")
        : "+v"(g.gx[0]), "+v"(g.gx[1]), "+v"(g.gx[2]), "=&v"(m0), "=&v"(m1), "=&v"(m2), "=&v"(m3)
        : "v"(o.d[0]), "v"(o.d[1]), "v"(o.d[2]), "v"(o.u[0]), "v"(o.u[1]), "v"(o.u[2]),
          "v"(o.Ab[0]), "v"(o.Ab[1]), "v"(o.Ab[2]), "v"(o.Bb[0]), "v"(o.Bb[1]), "v"(o.Bb[2]),
          "v"(o.r3), "v"(o.C1), "v"(o.C2), "v"(o.c3));
    asm("s_nop 1\n" NB_VJP_GU("0") NB_VJP_GU("1") NB_VJP_GU("2") NB_VJP_GU("3")
        : "+v"(g.gu[0]), "+v"(g.gu[1]), "+v"(g.gu[2]), "+v"(g.ngm), "=&v"(m0), "=&v"(m1), "=&v"(m2)
        : "v"(o.d[0]), "v"(o.d[1]), "v"(o.d[2]), "v"(o.Bb[0]), "v"(o.Bb[1]), "v"(o.Bb[2]),
          "v"(o.abq), "v"(o.bdq), "v"(o.r3), "v"(o.C2), "v"(o.c3));
}
#undef NB_VJP_GU
#undef NB_VJP_GX
#undef NB_F3
#undef NB_QUAD

// How a force VJP is split: i-blocks of ib rows with L lanes each times K ranges of tps j-tiles.
struct VjpPlan {
    int32_t L, ib, n_iblk, ntiles, tps, K, items;
    int64_t P;  // padded rows of one partial plane
};
// A lane's tile of 256 pairs is a serial chain (one wave issues an instruction every four cycles:
// 70 us whatever the size up to 16 tiles), so where the rows' lanes on all tiles leave the chip
// unfilled, rows take more: up to 64 slices in FP64 while they are at most four waves per SIMD
// (fill); in FP32, whose tile sums fix the slots' order, four helpers (vjp_add_quad, 177
// instructions per four pairs instead of 364, 108 of them half-rate DPP) up to 2/3 of that.
// With one lane and with more: N = 1000 FP32 75 and 37 us, FP64 71 and 17; N = 3276 77 and 72,
// 78 and 55; N = 4096 FP32 77 and 89 (hence the 2/3), FP64 81 and 68.
inline VjpPlan vjp_plan(int32_t n, bool fp32, int32_t num_cu, int32_t target) {
    VjpPlan p;
    p.ntiles = (n + TJ - 1) / TJ;
    const int64_t fill = (int64_t)num_cu * 1024 / p.ntiles;
    p.L = 1;
    if (fp32) {
        if ((int64_t)n * 6 <= fill) p.L = 4;
    } else {
        while (p.L < 64 && (int64_t)n * p.L * 2 <= fill) p.L *= 2;
    }
    p.ib = WG / p.L;
    p.n_iblk = (n + p.ib - 1) / p.ib;
    const int32_t K = std::max(1, std::min(target / p.n_iblk, p.ntiles));
    p.tps = (p.ntiles + K - 1) / K;
    p.K = (p.ntiles + p.tps - 1) / p.tps;
    p.items = p.n_iblk * p.K;
    p.P = (int64_t)p.n_iblk * p.ib;
    return p;
}

struct VjpArgs {
    int32_t n;
    const double *px, *py, *pz;  // predicted positions (FP64)
    const float4 *vm;            // FP32 mode: predicted velocity + mass
    const double *pm, *vx, *vy, *vz;  // FP64 mode
    const double *ab, *kb;       // adjoints of acc and jerk, 3 x n
    double eps2;
    double *partial;             // [K][7][P]
    VjpPlan pl;
};

template <class T>
struct VjpSmem {
    double x[TJ], y[TJ], z[TJ];
    T vx[TJ], vy[TJ], vz[TJ], m[TJ];
    T A[3][TJ], B[3][TJ];
};

template <int MODE>
using VjpT = typename std::conditional<MODE == 0, float, double>::type;

// Stages the j-particles of tile t (one per lane; padding carries zero mass and zero adjoints and
// adds exact zeros).
template <int MODE>
__device__ __forceinline__ void vjp_stage(const VjpArgs &a, VjpSmem<VjpT<MODE>> &sm, int32_t t) {
    using T = VjpT<MODE>;
    const int32_t n = a.n, x = threadIdx.x, j = t * TJ + x;
    const bool ok = j < n;
    const int32_t jc = ok ? j : 0;
    sm.x[x] = a.px[jc]; sm.y[x] = a.py[jc]; sm.z[x] = a.pz[jc];
    if (MODE == 0) {
        const float4 q = a.vm[jc];
        sm.vx[x] = q.x; sm.vy[x] = q.y; sm.vz[x] = q.z;
        sm.m[x] = ok ? q.w : 0.f;
    } else {
        sm.vx[x] = a.vx[jc]; sm.vy[x] = a.vy[jc];
        sm.vz[x] = a.vz[jc]; sm.m[x] = ok ? a.pm[jc] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        sm.A[k][x] = ok ? (T)a.ab[k * (int64_t)n + jc] : T(0);
        sm.B[k][x] = ok ? (T)a.kb[k * (int64_t)n + jc] : T(0);
    }
}

// Particle p of the force VJP: position, velocity, mass and negated adjoints.
template <class T>
struct VjpRow {
    double x, y, z;
    T vx, vy, vz, m, nA[3], nB[3];
};
template <int MODE>
__device__ __forceinline__ VjpRow<VjpT<MODE>> vjp_row(const VjpArgs &a, int32_t p) {
    using T = VjpT<MODE>;
    VjpRow<T> r;
    r.x = a.px[p]; r.y = a.py[p]; r.z = a.pz[p];
    if (MODE == 0) {
        const float4 q = a.vm[p];
        r.vx = q.x; r.vy = q.y; r.vz = q.z; r.m = q.w;
    } else {
        r.vx = a.vx[p]; r.vy = a.vy[p]; r.vz = a.vz[p]; r.m = a.pm[p];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.nA[k] = -(T)a.ab[k * (int64_t)a.n + p];
        r.nB[k] = -(T)a.kb[k * (int64_t)a.n + p];
        // opaque to the optimiser, which would otherwise fold the negation back into
        // modifiers on the products inside the pair loop
        asm volatile("" : "+v"(r.nA[k]), "+v"(r.nB[k]));
    }
    return r;
}

// The pair of row r with slot jj of the staged tile.  SOFT (eps > 0): every separation is
// positive, and only a tile holding the row's own slot (MASK, slot rel) needs a test; without
// softening every pair at zero separation (the self pair among them) adds nothing.
template <class T, bool SOFT, bool MASK>
__device__ __forceinline__ VjpTerms<T> vjp_slot(const VjpSmem<T> &sm, int32_t jj, int32_t rel,
                                                const VjpRow<T> &r, T eps2) {
    const T dx = (T)(sm.x[jj] - r.x), dy = (T)(sm.y[jj] - r.y), dz = (T)(sm.z[jj] - r.z);
    const T ux = sm.vx[jj] - r.vx, uy = sm.vy[jj] - r.vy, uz = sm.vz[jj] - r.vz;
    const T s = dx * dx + dy * dy + dz * dz + eps2;
    T rinv;
    if (std::is_same<T, float>::value) rinv = (T)__builtin_amdgcn_rsqf((float)s);
    else rinv = (T)rsqrt_f64((double)s);
    if (MASK && jj == rel) rinv = T(0);
    if (!SOFT && !(s > T(0))) rinv = T(0);
    const T Aq[3] = {sm.A[0][jj], sm.A[1][jj], sm.A[2][jj]};
    const T Bq[3] = {sm.B[0][jj], sm.B[1][jj], sm.B[2][jj]};
    return vjp_terms<T>(dx, dy, dz, ux, uy, uz, rinv, r.m, sm.m[jj], r.nA, r.nB, Aq, Bq);
}

// One staged tile for the lane `slice` of a row's L lanes: double takes every L-th slot; float,
// whose sums keep the slots' order, evaluates every fourth and adds all four lanes' (LANES: L
// is 4).  LANES = false: one lane a row.
template <class T, bool SOFT, bool MASK, bool LANES>
__device__ __forceinline__ void vjp_tile(const VjpSmem<T> &sm, int32_t slice, int32_t L,
                                         int32_t rel, const VjpRow<T> &r, T eps2, VjpSum<T> &g) {
    if constexpr (!LANES) {
#pragma unroll 1
        for (int jj = 0; jj < TJ; ++jj) g.add(vjp_slot<T, SOFT, MASK>(sm, jj, rel, r, eps2));
    } else if constexpr (std::is_same<T, float>::value) {
        for (int jj = slice; jj < TJ; jj += 4)
            vjp_add_quad(g, vjp_slot<T, SOFT, MASK>(sm, jj, rel, r, eps2));
    } else {
#pragma unroll 1
        for (int jj = slice; jj < TJ; jj += L) g.add(vjp_slot<T, SOFT, MASK>(sm, jj, rel, r, eps2));
    }
}

// Force VJP over all particles; j-split into K ranges, partial sums (7 per particle: x_bar,
// v_bar, m_bar) per range, summed by vjp_reduce.  MODE 0: float arithmetic on separations
// formed in double (tile sums folded into double); MODE 2: double throughout.  SOFT: eps > 0
// in the arithmetic type.  LANES: the plan gives a row more than one lane.
template <int MODE, bool SOFT, bool LANES>
__global__ void __launch_bounds__(WG) force_vjp_kernel(VjpArgs a) {
    using T = VjpT<MODE>;
    __shared__ VjpSmem<T> sm;
    const int32_t n = a.n;
    const VjpPlan &pl = a.pl;
    const int32_t L = LANES ? pl.L : 1, slice = LANES ? (int32_t)threadIdx.x & (L - 1) : 0;
    for (int32_t w = blockIdx.x; w < pl.items; w += gridDim.x) {
        const int32_t iblk = w / pl.K, ks = w - (w / pl.K) * pl.K;
        const int32_t p = LANES ? iblk * pl.ib + (int32_t)threadIdx.x / L
                                : iblk * WG + (int32_t)threadIdx.x;
        const int32_t own = p < n ? p : -1;  // p's own j-slot (none on padding lanes)
        const VjpRow<T> r = vjp_row<MODE>(a, p < n ? p : 0);
        double S[7] = {0, 0, 0, 0, 0, 0, 0};
        const T eps2 = (T)a.eps2;
        const int32_t t0 = ks * pl.tps;
        const int32_t t1 = t0 + pl.tps < pl.ntiles ? t0 + pl.tps : pl.ntiles;
        for (int32_t t = t0; t < t1; ++t) {
            __syncthreads();
            vjp_stage<MODE>(a, sm, t);
            __syncthreads();
            VjpSum<T> g;
            const int32_t rel = own - t * TJ;
            // a tile holding some lane's own slot takes the masked loop (wave-uniform branch)
            if (SOFT && __ballot((uint32_t)rel < (uint32_t)TJ) != 0)
                vjp_tile<T, SOFT, true, LANES>(sm, slice, L, rel, r, eps2, g);
            else
                vjp_tile<T, SOFT, false, LANES>(sm, slice, L, rel, r, eps2, g);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                S[k] += (double)g.gx[k];
                S[3 + k] += (double)g.gu[k];
            }
            S[6] -= (double)g.ngm;
        }
        if (LANES && MODE != 0) {  // the slices' sums (the four lanes of a float row hold the same)
            const auto swap_add = [&](auto off) {
                if (decltype(off)::value < L)
#pragma unroll
                    for (int k = 0; k < 7; ++k) S[k] += lane_xor<decltype(off)::value>(S[k]);
            };
            swap_add(std::integral_constant<int, 1>{});
            swap_add(std::integral_constant<int, 2>{});
            swap_add(std::integral_constant<int, 4>{});
            swap_add(std::integral_constant<int, 8>{});
            swap_add(std::integral_constant<int, 16>{});
            swap_add(std::integral_constant<int, 32>{});
        }
        if (p < n && slice == 0) {
            double *base = a.partial + (int64_t)ks * 7 * pl.P + p;
#pragma unroll
            for (int k = 0; k < 7; ++k) base[(int64_t)k * pl.P] = S[k];
        }
    }
}

// Sums the K partial planes (fixed order): x_bar, v_bar of the predicted state written to
// (accumulate = 0) or added to (accumulate = 1) xpb, vpb; m_bar added to mb.  Bound by the
// planes' bytes: one workgroup per (64 rows, one of the 7 sums), as force_reduce spreads them.
constexpr int VRW = WG / 64;
__global__ void __launch_bounds__(WG) vjp_reduce(int32_t n, const double *partial, VjpPlan pl,
                                                 double *xpb, double *vpb, double *mb,
                                                 int32_t accumulate) {
    __shared__ double part[VRW][64];
    const int32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t units = ((n + 63) >> 6) * 7;
    for (int32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int32_t rb = u / 7, c = u - rb * 7;
        const int32_t p = rb * 64 + lane;
        part[w][lane] = p < n ? wave_planes_sum<VRW>(partial + (int64_t)c * pl.P + p, 7 * pl.P, w, pl.K)
                              : 0.0;
        __syncthreads();
        if (w == 0 && p < n) {
            double t = part[0][lane];
#pragma unroll
            for (int r = 1; r < VRW; ++r) t += part[r][lane];
            double *o = c < 3 ? xpb + c * (int64_t)n + p
                      : c < 6 ? vpb + (c - 3) * (int64_t)n + p : mb + p;
            *o = (c == 6 || accumulate ? *o : 0.0) + t;
        }
        __syncthreads();
    }
}

}  // namespace nbody
