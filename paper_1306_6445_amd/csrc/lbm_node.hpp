// Arithmetic of one D2Q9 node, shared by every 2D step kernel: the inverse
// moment transform, the equilibrium moments, psi from the populations and the
// collision.  The same source expressions in all kernels give the same bits.
#pragma once

#include "lbm_device.hpp"

namespace lbm {

// f = M^-1 m for the orthogonal D2Q9 basis (rho, e, zeta, jx, qx, jy, qy, pxx, pxy):
// M^-1 = M^T diag(1/9, 1/36, 1/36, 1/6, 1/12, 1/6, 1/12, 1/4, 1/4).
// The conserved moments (rho, jx, jy) are not merely multiplied by a rounded
// reciprocal: 9 * fl(1/9) = 1 + 7.5e-9 in FP32, which would add mass at every
// step (1.5e-4 after 20,000 steps).  div_const corrects the product by its
// exact residual, which leaves no bias (the same mass drift as an IEEE
// division, at a third of the instructions).
template <typename C>
__device__ __forceinline__ void moments_to_pops(const C *m, C *f)
{
    const C a = div_const<C>(m[0], 9.0), b = m[1] * C(1.0 / 36.0), c = m[2] * C(1.0 / 36.0);
    const C d = div_const<C>(m[3], 6.0), e = m[4] * C(1.0 / 12.0), g = div_const<C>(m[5], 6.0);
    const C h = m[6] * C(1.0 / 12.0), i = m[7] * C(0.25), j = m[8] * C(0.25);
    const C ax = a - b - C(2) * c; // common part of the axis populations
    const C dg = a + C(2) * b + c; // common part of the diagonal populations
    f[0] = a - C(4) * b + C(4) * c;
    f[1] = ax + d - C(2) * e + i;
    f[2] = ax + g - C(2) * h - i;
    f[3] = ax - d + C(2) * e + i;
    f[4] = ax - g + C(2) * h - i;
    const C de = d + e, gh = g + h;
    f[5] = dg + de + gh + j;
    f[6] = dg - de + gh - j;
    f[7] = dg - de - gh + j;
    f[8] = dg + de - gh - j;
}

template <typename C>
__device__ __forceinline__ void equilibrium_moments(C rho, C vx, C vy, C *m)
{
    const C v2 = vx * vx + vy * vy;
    m[0] = rho;
    m[1] = rho * (C(-2) + C(3) * v2);
    m[2] = rho * (C(1) - C(3) * v2);
    m[3] = rho * vx;
    m[4] = -rho * vx;
    m[5] = rho * vy;
    m[6] = -rho * vy;
    m[7] = rho * (vx * vx - vy * vy);
    m[8] = rho * vx * vy;
}

// One node's collision: psi(x + e_a) from an LDS tile (lc points at psi(x),
// rows LX apart) and the pre-collision populations fv -> post-collision fs.
// MR: the multi-range force of Eq. (9), which also reads psi(x + 2 e_a).
// rho: the node's density, node_density(fv) (the collision conserves it).
template <typename C, bool MR = false>
__device__ __forceinline__ void collide_node(const RunPar<C> &k, const C *fv, C rho, const C *lc, int LX, C *fs)
{
    const C p0 = lc[0];
    const C p1 = lc[1], p3 = lc[-1], p2 = lc[LX], p4 = lc[-LX];
    const C p5 = lc[LX + 1], p6 = lc[LX - 1], p7 = lc[-LX - 1], p8 = lc[-LX + 1];

    const C G = k.G;
    // Eq. (7): F = -G psi(x) sum_a w_a psi(x + e_a) e_a, w = 1/3 (axis), 1/12 (diagonal)
    const C sx = C(1.0 / 3.0) * (p1 - p3) + C(1.0 / 12.0) * ((p5 - p7) + (p8 - p6));
    const C sy = C(1.0 / 3.0) * (p2 - p4) + C(1.0 / 12.0) * ((p5 - p7) + (p6 - p8));
    C Fx, Fy, F2; // F2 = |F|^2 / psi^2
    if constexpr (MR) {
        // Eq. (9): F = -psi(x) sum_a w_a [G1 psi(x + e_a) + G2 psi(x + 2 e_a)] e_a
        const int L2 = 2 * LX;
        const C q1 = lc[2], q3 = lc[-2], q2 = lc[L2], q4 = lc[-L2];
        const C q5 = lc[L2 + 2], q6 = lc[L2 - 2], q7 = lc[-L2 - 2], q8 = lc[-L2 + 2];
        const C tx = C(1.0 / 3.0) * (q1 - q3) + C(1.0 / 12.0) * ((q5 - q7) + (q8 - q6));
        const C ty = C(1.0 / 3.0) * (q2 - q4) + C(1.0 / 12.0) * ((q5 - q7) + (q6 - q8));
        const C G2 = k.G2;
        const C gx = G * sx + G2 * tx, gy = G * sy + G2 * ty;
        Fx = -p0 * gx;
        Fy = -p0 * gy;
        F2 = gx * gx + gy * gy;
    } else {
        Fx = -G * p0 * sx;
        Fy = -G * p0 * sy;
        F2 = G * G * (sx * sx + sy * sy);
    }
    // Eq. (19): Q = kappa G/2 psi(x) sum_a w_a [psi(x + e_a) - psi(x)] e_a e_a
    const C dsum = (p5 + p6) + (p7 + p8) - C(4) * p0;
    const C kq = k.kappa * G * C(0.5) * p0;
    const C Qxx = kq * (C(1.0 / 3.0) * (p1 + p3 - C(2) * p0) + C(1.0 / 12.0) * dsum);
    const C Qyy = kq * (C(1.0 / 3.0) * (p2 + p4 - C(2) * p0) + C(1.0 / 12.0) * dsum);
    const C Qxy = kq * (C(1.0 / 12.0) * ((p5 + p7) - (p6 + p8)));

    // Eq. (6): density (node_density, from the caller) and velocity (with F/2)
    const C sA = fv[1] + fv[3], sB = fv[2] + fv[4], sD = (fv[5] + fv[7]) + (fv[6] + fv[8]);
    const C d13 = fv[1] - fv[3], d24 = fv[2] - fv[4];
    const C d57 = fv[5] - fv[7], d86 = fv[8] - fv[6];
    const C jx = d13 + (d57 + d86);
    const C jy = d24 + (d57 - d86);
    const C irho = recip<C>(rho);
    const C vx = (jx + C(0.5) * Fx) * irho, vy = (jy + C(0.5) * Fy) * irho;

    // m = M f (non-conserved moments)
    const C sAB = sA + sB;
    const C m1 = C(-4) * fv[0] - sAB + C(2) * sD;
    const C m2 = C(4) * fv[0] - C(2) * sAB + sD;
    const C qdx = d57 + d86, qdy = d57 - d86;
    const C m4 = C(-2) * d13 + qdx;
    const C m6 = C(-2) * d24 + qdy;
    const C m7 = sA - sB;
    const C m8 = (fv[5] + fv[7]) - (fv[6] + fv[8]);

    // Eq. (3) equilibria
    const C vxx = vx * vx, vyy = vy * vy, v2 = vxx + vyy;
    const C e1 = rho * (C(-2) + C(3) * v2), e2 = rho * (C(1) - C(3) * v2);
    const C e7 = rho * (vxx - vyy), e8 = rho * vx * vy;

    // Eqs. (5), (8): S1 = 6 v.F + 12 sigma |F|^2 / (psi^2 (tau_e - 1/2));
    // |F|^2 / psi^2 = G^2 (sx^2 + sy^2) exactly (Eq. 7; F2 above).
    const C S1 = C(6) * (vx * Fx + vy * Fy) + k.sig_coef * F2;
    const C S7 = C(2) * (vx * Fx - vy * Fy);
    const C S8 = vx * Fy + vy * Fx;
    // Eq. (18)
    const C trQ = Qxx + Qyy;
    // Section V.C: the viscosity steps from nu_V to nu_L at the threshold density
    const C se = k.s_e, sz = k.s_zeta, sq = k.s_q;
    const C sv = rho < k.rho_nu ? k.s_nu_low : k.s_nu;
    const C C1 = C(1.5) * se * trQ, C2 = C(-1.5) * sz * trQ;
    const C C7 = -sv * (Qxx - Qyy), C8 = -sv * Qxy;

    // Eq. (17).  Conserved moments: m*_rho = rho, and with the Eq. (6) velocity
    // j* = j - s_j (j - rho v) + (1 - s_j/2) F = j + F for any s_j.
    C ms[9];
    ms[0] = rho;
    ms[1] = m1 - se * (m1 - e1) + (C(1) - C(0.5) * se) * S1 + C1;
    ms[2] = m2 - sz * (m2 - e2) - (C(1) - C(0.5) * sz) * S1 + C2;
    ms[3] = jx + Fx;
    ms[4] = m4 - sq * (m4 + rho * vx) - (C(1) - C(0.5) * sq) * Fx;
    ms[5] = jy + Fy;
    ms[6] = m6 - sq * (m6 + rho * vy) - (C(1) - C(0.5) * sq) * Fy;
    ms[7] = m7 - sv * (m7 - e7) + (C(1) - C(0.5) * sv) * S7 + C7;
    ms[8] = m8 - sv * (m8 - e8) + (C(1) - C(0.5) * sv) * S8 + C8;

    moments_to_pops<C>(ms, fs);
}

// psi of one node from its populations: the Eq. (6) density (node_density:
// compensated in FP32) and psi(rho) in the arithmetic type.  NaN and false
// where psi is not real.  rho_out receives the density.
template <typename C>
__device__ __forceinline__ bool node_psi(const RunPar<C> &k, int eos_kind, const C *fv, C &out, C &rho_out)
{
    const C rho = node_density<C>(fv);
    rho_out = rho;
    C ps;
    const bool ok = eval_psi<C>(k, eos_kind, rho, ps);
    out = ok ? ps : C(NAN);
    return ok;
}

} // namespace lbm
