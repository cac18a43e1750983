// HIP kernels (gfx950) of the two-component (binary mixture) extension of the
// pseudopotential MRT step with the surface-tension source term (Li & Luo,
// arXiv:1306.6445, Section VI names multicomponent models as future work; the
// two-component form follows the derivation in the design notes).  One step
// is one launch of mc_fused_kernel, or several are one of mc_multi_kernel:
//   each workgroup loads the populations of both components for its tile
//   (rows nodes per thread, ty rows apart) and a one-node ring around it,
//   sums the densities (psi_s = rho_s) into LDS, and after one barrier
//   collides every node of the tile: F_s (Eq. 7) and Q_s (Eq. 19) from the
//   other component's psi, the mixture velocity (Eq. 6 with both forces),
//   m_eq (Eq. 3) at rho_s and u, S (Eq. 5) with u and F_s, C (Eq. 18) with Q_s,
//   Eq. (17), f* = M^-1 m*, stored at the node in the second buffer.
// A buffer holds the post-collision state, streamed as it is read (Eq. 4;
// halfway bounce-back at walls: pull_slot2): loads are shifted by one node and
// stores aligned, which streams faster on this memory system than aligned
// loads with shifted stores.
#include <hip/hip_ext.h>

#include <type_traits>

#include "lbm3d_kernels.hpp"
#include "lbm_mc_kernels.hpp"
#include "lbm_multi.hpp"
#include "lbm_popbuf.hpp"

namespace lbmmc {

using lbm::ex_of;
using lbm::ey_of;
using lbm::opp_of;
using lbm3::AxisNb;
using lbm3::axis_nb;
using lbm3::nb_off;
using lbm3::nb_wall;

template <typename S> using ArithOf = typename std::conditional<std::is_same<S, double>::value, double, float>::type;

template <typename C> __device__ __forceinline__ C rate(const RunMC &r, int k)
{
    if constexpr (std::is_same<C, float>::value)
        return r.sf[k];
    else
        return r.s[k];
}

// FP32 storage: deviations f_a - w_a rho_ref[s] (the component's smallest
// initial density), decoded on load; FP64 stores the populations themselves.
template <typename C> __device__ __forceinline__ C ref_of(const RunMC &r, int s)
{
    if constexpr (std::is_same<C, float>::value)
        return r.rho_reff[s];
    else
        return C(0);
}
template <typename S, typename C> __device__ __forceinline__ C dec(S v, int a, C ref)
{
    if constexpr (std::is_same<S, double>::value)
        return v;
    else
        return v + C(lbm::rest_weight(a)) * ref;
}
template <typename S, typename C> __device__ __forceinline__ S enc(C v, int a, C ref)
{
    if constexpr (std::is_same<S, double>::value)
        return v;
    else
        return v - C(lbm::rest_weight(a)) * ref;
}

// f = M^-1 m for the orthogonal D2Q9 basis (the transform of the
// single-component kernels): M^-1 = M^T diag(1/9, 1/36, 1/36, 1/6, 1/12, 1/6,
// 1/12, 1/4, 1/4), the conserved moments divided with the FMA-residual
// correction so that FP32 adds no mass or momentum bias.
template <typename C> __device__ __forceinline__ void mc_moments_to_pops(const C *m, C *f)
{
    const C a = lbm::div_const<C>(m[0], 9.0), b = m[1] * C(1.0 / 36.0), c = m[2] * C(1.0 / 36.0);
    const C d = lbm::div_const<C>(m[3], 6.0), e = m[4] * C(1.0 / 12.0), g = lbm::div_const<C>(m[5], 6.0);
    const C h = m[6] * C(1.0 / 12.0), i = m[7] * C(0.25), j = m[8] * C(0.25);
    const C ax = a - b - C(2) * c, dg = a + C(2) * b + c;
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

// Eq. (7) and Eq. (19) on component s from the other component's psi p[a] =
// psi_o(x + e_a) (p[0] at x) and its own psi_s.
template <typename C>
__device__ __forceinline__ void force_q(C G, C kappa, C psi_s, const C *p, C &Fx, C &Fy, C &Qxx, C &Qyy, C &Qxy)
{
    const C sx = C(1.0 / 3.0) * (p[1] - p[3]) + C(1.0 / 12.0) * ((p[5] - p[7]) + (p[8] - p[6]));
    const C sy = C(1.0 / 3.0) * (p[2] - p[4]) + C(1.0 / 12.0) * ((p[5] - p[7]) + (p[6] - p[8]));
    Fx = -G * psi_s * sx;
    Fy = -G * psi_s * sy;
    const C dsum = (p[5] + p[6]) + (p[7] + p[8]) - C(4) * p[0];
    const C kq = kappa * G * C(0.5) * psi_s;
    Qxx = kq * (C(1.0 / 3.0) * (p[1] + p[3] - C(2) * p[0]) + C(1.0 / 12.0) * dsum);
    Qyy = kq * (C(1.0 / 3.0) * (p[2] + p[4] - C(2) * p[0]) + C(1.0 / 12.0) * dsum);
    Qxy = kq * (C(1.0 / 12.0) * ((p[5] + p[7]) - (p[6] + p[8])));
}

// One component's collision at one node: its populations fv and density rs,
// the mixture velocity (ux, uy), its force and source tensor -> fs.
template <typename C>
__device__ __forceinline__ void collide_mc(const RunMC &r, const C *fv, C rs, C ux, C uy, C Fx, C Fy, C Qxx, C Qyy,
                                           C Qxy, C *fs)
{
    const C se = rate<C>(r, 1), sz = rate<C>(r, 2), sj = rate<C>(r, 3), sq = rate<C>(r, 4), sv = rate<C>(r, 7);
    const C sA = fv[1] + fv[3], sB = fv[2] + fv[4], sD = (fv[5] + fv[7]) + (fv[6] + fv[8]);
    const C d13 = fv[1] - fv[3], d24 = fv[2] - fv[4], d57 = fv[5] - fv[7], d86 = fv[8] - fv[6];
    const C jx = d13 + (d57 + d86), jy = d24 + (d57 - d86);
    const C sAB = sA + sB;
    const C m1 = C(-4) * fv[0] - sAB + C(2) * sD;
    const C m2 = C(4) * fv[0] - C(2) * sAB + sD;
    const C m4 = C(-2) * d13 + (d57 + d86), m6 = C(-2) * d24 + (d57 - d86);
    const C m7 = sA - sB, m8 = (fv[5] + fv[7]) - (fv[6] + fv[8]);
    // Eq. (3) at the component's density and the mixture velocity
    const C uxx = ux * ux, uyy = uy * uy, u2 = uxx + uyy;
    const C e1 = rs * (C(-2) + C(3) * u2), e2 = rs * (C(1) - C(3) * u2);
    const C e7 = rs * (uxx - uyy), e8 = rs * ux * uy;
    // Eq. (5) with the mixture velocity and the component's force
    const C S1 = C(6) * (ux * Fx + uy * Fy), S7 = C(2) * (ux * Fx - uy * Fy), S8 = ux * Fy + uy * Fx;
    // Eq. (18) with the component's Q
    const C trQ = Qxx + Qyy;
    const C C1 = C(1.5) * se * trQ, C2 = C(-1.5) * sz * trQ, C7 = -sv * (Qxx - Qyy), C8 = -sv * Qxy;
    // Eq. (17); the component's momentum relaxes toward rho_s u (inter-diffusion)
    C ms[9];
    ms[0] = rs;
    ms[1] = m1 - se * (m1 - e1) + (C(1) - C(0.5) * se) * S1 + C1;
    ms[2] = m2 - sz * (m2 - e2) - (C(1) - C(0.5) * sz) * S1 + C2;
    ms[3] = jx - sj * (jx - rs * ux) + (C(1) - C(0.5) * sj) * Fx;
    ms[4] = m4 - sq * (m4 + rs * ux) - (C(1) - C(0.5) * sq) * Fx;
    ms[5] = jy - sj * (jy - rs * uy) + (C(1) - C(0.5) * sj) * Fy;
    ms[6] = m6 - sq * (m6 + rs * uy) - (C(1) - C(0.5) * sq) * Fy;
    ms[7] = m7 - sv * (m7 - e7) + (C(1) - C(0.5) * sv) * S7 + C7;
    ms[8] = m8 - sv * (m8 - e8) + (C(1) - C(0.5) * sv) * S8 + C8;
    mc_moments_to_pops<C>(ms, fs);
}

// Both components of one node: populations fA, fB with densities rA, rB, the
// densities pA, pB of the node and its neighbours -> post-collision sa, sb.
template <typename C>
__device__ __forceinline__ void collide_both(const RunMC &r, C G, C kappa, const C *fA, const C *fB, C rA, C rB,
                                             const C *pA, const C *pB, C *sa, C *sb)
{
    // psi_s = rho_s: A feels B's psi and B feels A's
    C FAx, FAy, QAxx, QAyy, QAxy, FBx, FBy, QBxx, QByy, QBxy;
    force_q<C>(G, kappa, rA, pB, FAx, FAy, QAxx, QAyy, QAxy);
    force_q<C>(G, kappa, rB, pA, FBx, FBy, QBxx, QByy, QBxy);
    // Eq. (6) for the mixture
    C jx = C(0), jy = C(0);
#pragma unroll
    for (int a = 1; a < 9; ++a) {
        const C v = fA[a] + fB[a];
        if (ex_of(a)) jx += C(ex_of(a)) * v;
        if (ey_of(a)) jy += C(ey_of(a)) * v;
    }
    const C irho = lbm::recip<C>(rA + rB);
    const C ux = (jx + C(0.5) * (FAx + FBx)) * irho, uy = (jy + C(0.5) * (FAy + FBy)) * irho;
    collide_mc<C>(r, fA, rA, ux, uy, FAx, FAy, QAxx, QAyy, QAxy, sa);
    collide_mc<C>(r, fB, rB, ux, uy, FBx, FBy, QBxx, QByy, QBxy, sb);
}

// streamed populations of both components of node n (host-order index
// y nx + x, neighbour offsets X, Y)
template <typename S, typename C>
__device__ __forceinline__ void gather18(const S *__restrict__ f, int64_t N, int64_t n, const AxisNb &X,
                                         const AxisNb &Y, C refA, C refB, C *fa, C *fb)
{
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const int64_t i = pull_slot2(n, X, Y, a, N);
        fa[a] = dec<S, C>(f[i], a, refA);
        fb[a] = dec<S, C>(f[9 * N + i], a, refB);
    }
}

// The same read for a buffer of less than 4 GiB: every slot's byte offset
// from the buffer's start fits in 32 bits, so each load takes one offset
// register beside the buffer's scalar base.  Offsets wrap modulo 2^32 and the
// final offset is exact.
template <typename S, typename C>
__device__ __forceinline__ void gather18_w32(const S *__restrict__ f, uint32_t N, uint32_t n, const AxisNb &X,
                                             const AxisNb &Y, C refA, C refB, C *fa, C *fb)
{
    const char *base = reinterpret_cast<const char *>(f);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const bool wall = nb_wall(X, -ex_of(a)) || nb_wall(Y, -ey_of(a));
        const uint32_t i = wall ? (uint32_t)opp_of(a) * N + n
                                : (uint32_t)a * N + n + (uint32_t)nb_off(X, -ex_of(a)) + (uint32_t)nb_off(Y, -ey_of(a));
        fa[a] = dec<S, C>(*reinterpret_cast<const S *>(base + (uint32_t)(i * (uint32_t)sizeof(S))), a, refA);
        fb[a] = dec<S, C>(*reinterpret_cast<const S *>(base + (uint32_t)((9 * N + i) * (uint32_t)sizeof(S))), a, refB);
    }
}

template <typename S, typename C, bool W32>
__device__ __forceinline__ void gather18_at(const S *__restrict__ f, int64_t N, int64_t n, const AxisNb &X,
                                            const AxisNb &Y, C refA, C refB, C *fa, C *fb)
{
    if constexpr (W32)
        gather18_w32<S, C>(f, (uint32_t)N, (uint32_t)n, X, Y, refA, refB, fa, fb);
    else
        gather18<S, C>(f, N, n, X, Y, refA, refB, fa, fb);
}

template <typename S, int R, bool W32>
__global__ void __launch_bounds__(512) mc_fused_kernel(const RunMC *__restrict__ runs, const S *__restrict__ fin,
                                                       S *__restrict__ fout, int32_t *__restrict__ status)
{
    using C = ArithOf<S>;
    extern __shared__ unsigned char lds_raw[];
    const RunMC &r = runs[0];
    const int nx = r.nx, ny = r.ny, bcx = r.bc_x, bcy = r.bc_y;
    const int TX = blockDim.x, TY = blockDim.y, TYR = R * TY, LX = TX + 2, LY = TYR + 2;
    C *la = reinterpret_cast<C *>(lds_raw);
    C *lb = la + LX * LY;
    int x0, y0;
    mc_tile_origin(lbm::work_index(1), nx, TX, TY, R, x0, y0);
    const int64_t N = r.dstride;
    const C refA = ref_of<C>(r, 0), refB = ref_of<C>(r, 1);
    bool bad = false;

    // the tile's own nodes (a column beyond the grid edge fills its LDS cell
    // with the wrapped or clamped node and collides nothing)
    const int x = x0 + (int)threadIdx.x;
    const int gx = lbm::psi_coord(x, nx, bcx);
    const AxisNb GX = axis_nb(gx, nx, bcx, 1);
    C fA[R][9], fB[R][9], rA[R], rB[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int y = y0 + (int)threadIdx.y + j * TY;
        const int gy = lbm::psi_coord(y, ny, bcy);
        gather18_at<S, C, W32>(fin, N, (int64_t)gy * nx + gx, GX, axis_nb(gy, ny, bcy, nx), refA, refB, fA[j], fB[j]);
        rA[j] = lbm::node_density<C>(fA[j]);
        rB[j] = lbm::node_density<C>(fB[j]);
        bad |= !(rA[j] + rB[j] > C(0)) || !(rA[j] - rA[j] == C(0)) || !(rB[j] - rB[j] == C(0));
        const int cell = ((int)threadIdx.y + j * TY + 1) * LX + (int)threadIdx.x + 1;
        la[cell] = rA[j];
        lb[cell] = rB[j];
    }
    // densities of the one-node ring: rows 0 and LY - 1 of the LDS tile, then columns 0 and LX - 1
    const int nring = 2 * LX + 2 * TYR;
    for (int k = (int)(threadIdx.y * TX + threadIdx.x); k < nring; k += TX * TY) {
        int lx, ly;
        mc_ring_cell(k, LX, LY, lx, ly);
        const int hx = lbm::psi_coord(x0 - 1 + lx, nx, bcx), hy = lbm::psi_coord(y0 - 1 + ly, ny, bcy);
        C ha[9], hb[9];
        gather18_at<S, C, W32>(fin, N, (int64_t)hy * nx + hx, axis_nb(hx, nx, bcx, 1), axis_nb(hy, ny, bcy, nx), refA,
                               refB, ha, hb);
        const C da = lbm::node_density<C>(ha), db = lbm::node_density<C>(hb);
        bad |= !(da + db > C(0)) || !(da - da == C(0)) || !(db - db == C(0));
        la[ly * LX + lx] = da;
        lb[ly * LX + lx] = db;
    }
    if (bad) status[0] = 1;
    __syncthreads();
    if (x >= nx) return;

    const C G = std::is_same<C, float>::value ? C(r.Gf) : C(r.G);
    const C kappa = std::is_same<C, float>::value ? C(r.kappaf) : C(r.kappa);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int y = y0 + (int)threadIdx.y + j * TY;
        if (y >= ny) break;
        const int cell = ((int)threadIdx.y + j * TY + 1) * LX + (int)threadIdx.x + 1;
        C pA[9], pB[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            pA[a] = la[cell + ey_of(a) * LX + ex_of(a)];
            pB[a] = lb[cell + ey_of(a) * LX + ex_of(a)];
        }
        C sa[9], sb[9];
        collide_both<C>(r, G, kappa, fA[j], fB[j], rA[j], rB[j], pA, pB, sa, sb);
        // f* stays at the node; the next read streams it (Eq. 4)
        const int64_t n = (int64_t)y * nx + x;
        if constexpr (W32) {
            char *base = reinterpret_cast<char *>(fout);
            const uint32_t N32 = (uint32_t)N, n32 = (uint32_t)n;
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                *reinterpret_cast<S *>(base + (uint32_t)(((uint32_t)a * N32 + n32) * (uint32_t)sizeof(S))) =
                    enc<S, C>(sa[a], a, refA);
                *reinterpret_cast<S *>(base + (uint32_t)(((uint32_t)(9 + a) * N32 + n32) * (uint32_t)sizeof(S))) =
                    enc<S, C>(sb[a], a, refB);
            }
        } else {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                fout[(int64_t)a * N + n] = enc<S, C>(sa[a], a, refA);
                fout[(int64_t)(9 + a) * N + n] = enc<S, C>(sb[a], a, refB);
            }
        }
    }
}

// Several steps in one launch, the intermediate states in LDS (see
// lbm_multi.hpp): step s of K collides the tile and a margin of 2 (K - s) nodes.
// The state is f*_a at the node, streamed on the read, so the first step gathers
// from the source buffer, the later ones from LDS and the last stores at the
// node.  The intermediate state passes through LDS in its storage form: the same
// bits as single steps.
//
// What bounds it: the single step moved 149 B of counted traffic a node and step
// (FP32) at 4.4-4.9 TB/s; two steps a launch halve that, and vector issue, with
// the margins done again by the neighbours, bounds the rest.  us per step, one ->
// several a launch: 2048^2 FP32 127 -> 100, FP64 244 -> 194; 1300^2 FP32 34.7, FP64 81.3;
// 100^2 FP32 5.1 -> 2.9, FP64 6.4 -> 3.2.
template <typename S, int K, int TX, int TY, int NT, bool WALLS> struct MultiMC {
    using C = ArithOf<S>;
    using Gm = lbm::MultiGeom<K, TX, TY>;
    const RunMC &r;
    const int nx, ny, bcx, bcy, x0, y0;
    const uint32_t ds; // bytes from one direction's array to the next
    const C refA, refB, G, kappa;
    const lbm::PopBuf<S> in, out;
    C *la, *lb; // densities
    S *pop;     // component A's nine planes of FN cells, then component B's
    bool bad = false;

    template <int s> __device__ __forceinline__ void load(int dx, int dy, C *fa, C *fb) const
    {
        const int gx = lbm::psi_coord(x0 + dx, nx, WALLS ? bcx : lbm::BC_PERIODIC);
        const int gy = lbm::psi_coord(y0 + dy, ny, WALLS ? bcy : lbm::BC_PERIODIC);
        const lbm::Nbr n = lbm::neighbours(gx, gy, nx, ny, WALLS ? bcx : lbm::BC_PERIODIC, WALLS ? bcy : lbm::BC_PERIODIC);
        auto wall = [&](int a) {
            const int ex = ex_of(a), ey = ey_of(a);
            return WALLS && ((ex > 0 && n.wxm) || (ex < 0 && n.wxp) || (ey > 0 && n.wym) || (ey < 0 && n.wyp));
        };
        if constexpr (s == 1) {
            constexpr uint32_t z = sizeof(S);
            const uint32_t xo[3] = {n.xm * z, gx * z, n.xp * z};
            const uint32_t yo[3] = {n.ym * nx * z, gy * nx * z, n.yp * nx * z};
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const uint32_t up = xo[1 - ex_of(a)] + yo[1 - ey_of(a)];
                if constexpr (WALLS) {
                    const uint32_t i = wall(a) ? opp_of(a) * ds + xo[1] + yo[1] : a * ds + up;
                    fa[a] = dec<S, C>(in.load(i, 0), a, refA);
                    fb[a] = dec<S, C>(in.load(i, 9 * ds), a, refB);
                } else {
                    fa[a] = dec<S, C>(in.load(up, a * ds), a, refA);
                    fb[a] = dec<S, C>(in.load(up, (9 + a) * ds), a, refB);
                }
            }
        } else {
            // LDS cell: unwrapped on a periodic axis, the clamped node's across a wall
            const int cx = WALLS && bcx == lbm::BC_WALL ? gx - x0 : dx, cy = WALLS && bcy == lbm::BC_WALL ? gy - y0 : dy;
            const int cell = Gm::pop(cx, cy);
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const int i = Gm::pull(a, cell, wall(a));
                fa[a] = dec<S, C>(pop[i], a, refA);
                fb[a] = dec<S, C>(pop[9 * Gm::FN + i], a, refB);
            }
        }
    }

    __device__ __forceinline__ void put(int dx, int dy, const C *fa, const C *fb, C &da, C &db)
    {
        da = lbm::node_density<C>(fa);
        db = lbm::node_density<C>(fb);
        bad |= !(da + db > C(0)) || !(da - da == C(0)) || !(db - db == C(0));
        const int cell = Gm::psi(dx, dy);
        la[cell] = da;
        lb[cell] = db;
    }

    template <int s> __device__ __forceinline__ void step(int tid)
    {
        constexpr int N = Gm::cells(s), NI = N + Gm::ring(s), R = (N + NT - 1) / NT;
        C fA[R][9], fB[R][9], rA[R], rB[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT;
            if (i < NI) {
                int dx, dy;
                lbm::multi_item<Gm, s, K>(i, dx, dy);
                load<s>(dx, dy, fA[j], fB[j]);
                put(dx, dy, fA[j], fB[j], rA[j], rB[j]);
            }
        }
        for (int i = tid + R * NT; i < NI; i += NT) {
            int dx, dy;
            lbm::multi_item<Gm, s, K>(i, dx, dy);
            C ha[9], hb[9], da, db;
            load<s>(dx, dy, ha, hb);
            put(dx, dy, ha, hb, da, db);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT;
            if (i < N) {
                const int ly = (unsigned)i / (unsigned)Gm::w(s), lx = i - ly * Gm::w(s);
                const int dx = lx - 2 * (K - s), dy = ly - 2 * (K - s);
                const int cell = (dy + Gm::M + 1) * Gm::PX + dx + Gm::M + 1;
                C pA[9], pB[9], sa[9], sb[9];
#pragma unroll
                for (int a = 0; a < 9; ++a) {
                    pA[a] = la[cell + ey_of(a) * Gm::PX + ex_of(a)];
                    pB[a] = lb[cell + ey_of(a) * Gm::PX + ex_of(a)];
                }
                collide_both<C>(r, G, kappa, fA[j], fB[j], rA[j], rB[j], pA, pB, sa, sb);
                if constexpr (s < K) {
                    const int q = (dy + Gm::M) * Gm::FX + dx + Gm::M;
#pragma unroll
                    for (int a = 0; a < 9; ++a) {
                        pop[a * Gm::FN + q] = enc<S, C>(sa[a], a, refA);
                        pop[(9 + a) * Gm::FN + q] = enc<S, C>(sb[a], a, refB);
                    }
                } else {
                    const int x = x0 + dx, y = y0 + dy;
                    if (x < nx && y < ny) {
                        const uint32_t off = (uint32_t)(y * nx + x) * (uint32_t)sizeof(S);
#pragma unroll
                        for (int a = 0; a < 9; ++a) {
                            out.store(off, a * ds, enc<S, C>(sa[a], a, refA));
                            out.store(off, (9 + a) * ds, enc<S, C>(sb[a], a, refB));
                        }
                    }
                }
            }
        }
        if constexpr (s < K) {
            __syncthreads();
            step<s + 1>(tid);
        }
    }
};

template <typename S, int K, int TX, int TY, int NT>
__global__ void __launch_bounds__(NT) mc_multi_kernel(const RunMC *__restrict__ runs, const S *__restrict__ fin,
                                                      S *__restrict__ fout, int32_t *__restrict__ status)
{
    using C = ArithOf<S>;
    using Gm = lbm::MultiGeom<K, TX, TY>;
    __shared__ C la[Gm::PN], lb[Gm::PN];
    __shared__ S pop[18 * Gm::FN];
    const RunMC &r = runs[0];
    const int ntx = (r.nx + TX - 1) / TX, wi = lbm::work_index(1), x0 = wi % ntx * TX, y0 = wi / ntx * TY;
    const uint32_t ds = (uint32_t)r.dstride * (uint32_t)sizeof(S);
    const C G = std::is_same<C, float>::value ? C(r.Gf) : C(r.G);
    const C kappa = std::is_same<C, float>::value ? C(r.kappaf) : C(r.kappa);
    // reach of the first step's reads beyond the tile
    constexpr int E = Gm::M + 2;
    const bool free_x = r.bc_x == lbm::BC_PERIODIC || (x0 >= E && x0 + TX + E <= r.nx);
    const bool free_y = r.bc_y == lbm::BC_PERIODIC || (y0 >= E && y0 + TY + E <= r.ny);
    bool bad;
    if (free_x && free_y) {
        MultiMC<S, K, TX, TY, NT, false> m{r, r.nx, r.ny, r.bc_x, r.bc_y, x0, y0, ds, ref_of<C>(r, 0), ref_of<C>(r, 1), G,
                                          kappa, lbm::PopBuf<S>(fin), lbm::PopBuf<S>(fout), la, lb, pop};
        m.template step<1>((int)threadIdx.x);
        bad = m.bad;
    } else {
        MultiMC<S, K, TX, TY, NT, true> m{r, r.nx, r.ny, r.bc_x, r.bc_y, x0, y0, ds, ref_of<C>(r, 0), ref_of<C>(r, 1), G,
                                         kappa, lbm::PopBuf<S>(fin), lbm::PopBuf<S>(fout), la, lb, pop};
        m.template step<1>((int)threadIdx.x);
        bad = m.bad;
    }
    if (bad) status[0] = 1;
}

// ------------------------------------------------------------- utilities

template <typename S>
__global__ void __launch_bounds__(kThreadsMC) util_mc_kernel(const RunMC *__restrict__ runs, int op,
                                                             const S *__restrict__ fin, S *__restrict__ fout,
                                                             double *__restrict__ buf)
{
    using C = ArithOf<S>;
    const RunMC &r = runs[0];
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t NN = r.nodes, N = r.dstride;
    if (n >= NN) return;
    const C ref[2] = {ref_of<C>(r, 0), ref_of<C>(r, 1)};
    const int x = (int)(n % r.nx), y = (int)(n / r.nx);
    const AxisNb X = axis_nb(x, r.nx, r.bc_x, 1), Y = axis_nb(y, r.ny, r.bc_y, r.nx);
    // slot of the streamed population f_a(x) of component s (reads), and
    // where a state given as f_a(x) goes (writes: each slot once)
    auto slot = [&](int s, int a) { return (int64_t)s * 9 * N + pull_slot2(n, X, Y, a, N); };
    if (op == 0) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int a = 0; a < 9; ++a)
                buf[(int64_t)(s * 9 + a) * NN + n] = (double)dec<S, C>(fin[slot(s, a)], a, ref[s]);
    } else if (op == 1) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int a = 0; a < 9; ++a) fout[slot(s, a)] = enc<S, C>((C)buf[(int64_t)(s * 9 + a) * NN + n], a, ref[s]);
    } else if (op == 2) {
        // f = M^-1 m_eq(rho_s, u) (Eq. 3), in FP64 then rounded to the storage
        const double ux = buf[2 * NN + n], uy = buf[3 * NN + n], u2 = ux * ux + uy * uy;
        for (int s = 0; s < 2; ++s) {
            const double rho = buf[s * NN + n];
            const double m[9] = {rho, rho * (-2.0 + 3.0 * u2), rho * (1.0 - 3.0 * u2), rho * ux, -rho * ux,
                                 rho * uy, -rho * uy, rho * (ux * ux - uy * uy), rho * ux * uy};
            double fd[9];
            mc_moments_to_pops<double>(m, fd);
#pragma unroll
            for (int a = 0; a < 9; ++a) fout[slot(s, a)] = enc<S, C>((C)fd[a], a, ref[s]);
        }
    } else if (op == 3) {
        for (int s = 0; s < 2; ++s) {
            double rho = 0.0;
#pragma unroll
            for (int a = 0; a < 9; ++a) rho += (double)dec<S, C>(fin[slot(s, a)], a, ref[s]);
            buf[s * NN + n] = rho;
        }
    } else {
        // Eq. (6) for the mixture, FP64, from the densities in buf[0, 2N)
        double pA[9], pB[9];
        for (int a = 0; a < 9; ++a) {
            const int64_t m = (int64_t)lbm::psi_coord(y + ey_of(a), r.ny, r.bc_y) * r.nx +
                              lbm::psi_coord(x + ex_of(a), r.nx, r.bc_x);
            pA[a] = buf[m];
            pB[a] = buf[NN + m];
        }
        double FAx, FAy, FBx, FBy, q0, q1, q2;
        force_q<double>(r.G, 0.0, pA[0], pB, FAx, FAy, q0, q1, q2);
        force_q<double>(r.G, 0.0, pB[0], pA, FBx, FBy, q0, q1, q2);
        double jx = 0.0, jy = 0.0;
        for (int s = 0; s < 2; ++s)
            for (int a = 1; a < 9; ++a) {
                const double v = (double)dec<S, C>(fin[slot(s, a)], a, ref[s]);
                jx += ex_of(a) * v;
                jy += ey_of(a) * v;
            }
        const double rho = pA[0] + pB[0];
        buf[2 * NN + n] = (jx + 0.5 * (FAx + FBx)) / rho;
        buf[3 * NN + n] = (jy + 0.5 * (FAy + FBy)) / rho;
    }
}

__global__ void __launch_bounds__(kThreadsMC) diag_mc_kernel(const RunMC *__restrict__ runs,
                                                             const double *__restrict__ buf, double cx, double cy,
                                                             double r_in, double r_out, double *__restrict__ partial)
{
    __shared__ double red[kDiagMC][kThreadsMC];
    const RunMC &r = runs[0];
    const int64_t NN = r.nodes, n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int tid = threadIdx.x;
    double v[kDiagMC] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (n < NN) {
        const double a = buf[n], b = buf[NN + n], ux = buf[2 * NN + n], uy = buf[3 * NN + n];
        const int x = (int)(n % r.nx), y = (int)(n / r.nx);
        double dx = x - cx, dy = y - cy;
        if (r.bc_x == lbm::BC_PERIODIC) dx -= r.nx * rint(dx / r.nx);
        if (r.bc_y == lbm::BC_PERIODIC) dy -= r.ny * rint(dy / r.ny);
        const double dist = sqrt(dx * dx + dy * dy);
        // bulk pressure of the mixture: (rho_A + rho_B) / 3 + G rho_A rho_B
        const double p = (a + b) / 3.0 + r.G * a * b;
        v[0] = a;
        v[1] = b;
        if (dist <= r_in) {
            v[2] = a;
            v[3] = b;
            v[4] = 1.0;
            v[8] = p;
        }
        if (dist >= r_out) {
            v[5] = a;
            v[6] = b;
            v[7] = 1.0;
            v[9] = p;
        }
        const double sp = sqrt(ux * ux + uy * uy);
        v[10] = sp == sp ? sp : INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kDiagMC; ++q) red[q][tid] = v[q];
    __syncthreads();
    for (int s = kThreadsMC / 2; s > 0; s >>= 1) {
        if (tid < s) {
#pragma unroll
            for (int q = 0; q < kDiagMC - 1; ++q) red[q][tid] += red[q][tid + s];
            red[kDiagMC - 1][tid] = fmax(red[kDiagMC - 1][tid], red[kDiagMC - 1][tid + s]);
        }
        __syncthreads();
    }
    if (tid < kDiagMC) partial[(int64_t)blockIdx.x * kDiagMC + tid] = red[tid][0];
}

// ------------------------------------------------------------- launchers

template <typename S, int R> hipError_t fused_mc_t(const StepMCArgs &a)
{
    using C = ArithOf<S>;
    const uint32_t lds = 2 * sizeof(C) * (a.tx + 2) * (R * a.ty + 2);
    const int64_t tiles = mc_tiles(a.nx, a.ny, a.tx, a.ty, R);
    if (a.w32)
        hipExtLaunchKernelGGL((mc_fused_kernel<S, R, true>), dim3((unsigned)tiles), dim3(a.tx, a.ty), lds, a.stream,
                              a.ev0, a.ev1, 0, a.run, static_cast<const S *>(a.fin), static_cast<S *>(a.fout), a.status);
    else
        hipExtLaunchKernelGGL((mc_fused_kernel<S, R, false>), dim3((unsigned)tiles), dim3(a.tx, a.ty), lds, a.stream,
                              a.ev0, a.ev1, 0, a.run, static_cast<const S *>(a.fin), static_cast<S *>(a.fout), a.status);
    return hipGetLastError();
}

template <typename S> hipError_t step_mc_t(const StepMCArgs &a)
{
    switch (a.rows) {
    case 1: return fused_mc_t<S, 1>(a);
    case 4: return fused_mc_t<S, 4>(a);
    default: return fused_mc_t<S, 2>(a);
    }
}

hipError_t launch_step_mc(int precision, const StepMCArgs &a)
{
    if (!mc_shape_ok(a.tx, a.ty, a.rows)) return hipErrorInvalidValue;
    return precision == PRECMC_FP64 ? step_mc_t<double>(a) : step_mc_t<float>(a);
}

namespace {

template <typename S, int K, int TX, int TY, int NT> hipError_t launch_multi_mc_t(const StepMCArgs &a)
{
    const lbm::MultiShape shape{K, TX, TY};
    const dim3 grid((unsigned)lbm::multi_tiles(shape, a.nx, a.ny));
    hipExtLaunchKernelGGL((mc_multi_kernel<S, K, TX, TY, NT>), grid, dim3(NT), 0, a.stream, a.ev0, a.ev1, 0, a.run,
                          static_cast<const S *>(a.fin), static_cast<S *>(a.fout), a.status);
    return hipGetLastError();
}

struct VariantMC {
    lbm::MultiShape shape;
    double work;       // relative vector work of a tile: 130 a cell's densities, 440 a collision
    int64_t max_tiles; // small tiles: taken when the grid has no more of them than this
    hipError_t (*launch)(const StepMCArgs &);
};

template <typename S, int K, int TX, int TY, int NT> constexpr VariantMC variant_of(int64_t max_tiles)
{
    using Gm = lbm::MultiGeom<K, TX, TY>;
    double work = 0.0;
    for (int s = 1; s <= K; ++s) work += 130.0 * (Gm::cells(s) + Gm::ring(s)) + 440.0 * Gm::cells(s);
    return {{K, TX, TY}, work, max_tiles, launch_multi_mc_t<S, K, TX, TY, NT>};
}

// 72 (FP32) or 144 bytes of LDS a cell keep the tiles small.  Small grids take
// the tile with the shortest chain (us a step, FP32: 100^2 2.9 with 8 x 8 and K =
// 4 against 4.0 with 28 x 12 and 5.1 one step at a time; 400^2 6.2 with 28 x 12
// against 6.7 with 32 x 16), the others the largest tile that leaves two
// workgroups a CU and fills the rounds of its threads, with rows that start on
// 128 bytes (FP32, us a step: 1300^2 34.9 with 32 x 24 against 38.2 with 64 x 8 and
// 37.3 with 28 x 24, 2048^2 101.7 / 102.0 / 99.7; FP64 1300^2 82.0 with 32 x 8
// against 86.4 with 28 x 8, 2048^2 195 / 201).
const VariantMC kMc32[] = {
    variant_of<float, 4, 8, 8, 512>(256),
    variant_of<float, 2, 28, 12, 512>(768),
    variant_of<float, 2, 32, 24, 768>(0),
};
const VariantMC kMc64[] = {
    variant_of<double, 4, 8, 8, 512>(256),
    variant_of<double, 2, 32, 8, 512>(0),
};

const VariantMC *variant_mc(int precision, int v)
{
    if (precision == PRECMC_FP32) return v >= 0 && v < (int)(sizeof(kMc32) / sizeof(kMc32[0])) ? &kMc32[v] : nullptr;
    return v >= 0 && v < (int)(sizeof(kMc64) / sizeof(kMc64[0])) ? &kMc64[v] : nullptr;
}

} // namespace

// Besides the shapes' own rules, single steps (of tx x ty threads, `rows` nodes
// each) stay where the tiles' rows beyond a flat grid cost more than the launches
// save: when the tiles outnumber the resident workgroups, two a CU, several steps a
// launch are taken up to 2.6 times the work of as many single steps (waves beyond
// the grid's last row or column do none).  Measured, us a step, single against
// several: FP32 at 1.3 times the work 100000 x 20 65.9 / 48.4, at 2.1 100000 x 12 37.9 /
// 37.0, at 3.2 200000 x 8 47.8 / 60.5, at 6.4 400000 x 4 41.9 / 102; FP64 at 2.5 400000
// x 4 114 / 93, at 7.5 100000 x 1 17.1 / 22.1.
int pick_multi_mc(int precision, int nx, int ny, int tx, int ty, int rows, lbm::MultiShape &shape)
{
    int best = -1;
    double least = 0.0;
    for (int v = 0; const VariantMC *p = variant_mc(precision, v); ++v) {
        const int64_t tiles = lbm::multi_tiles(p->shape, nx, ny);
        if (p->max_tiles > 0 && tiles > p->max_tiles) continue;
        if (p->max_tiles > 0 || best < 0 || (double)tiles * p->work < least) {
            best = v;
            least = (double)tiles * p->work;
            shape = p->shape;
        }
        if (p->max_tiles > 0) break;
    }
    const int wide = tx < 64 ? tx : 64, high = ty * rows;
    const double single = (double)((nx + wide - 1) / wide * wide) * ny * (130.0 + 440.0) +
                          (double)lbm::multi_tiles({1, tx, high}, nx, ny) * 130.0 * (2 * (tx + 2) + 2 * high);
    return lbm::multi_tiles(shape, nx, ny) > 512 && least > 2.6 * shape.steps * single ? -1 : best;
}

hipError_t launch_multi_mc(int precision, int v, const StepMCArgs &a)
{
    const VariantMC *p = variant_mc(precision, v);
    return p && a.w32 ? p->launch(a) : hipErrorInvalidValue;
}

static unsigned blocks_mc(int64_t n) { return (unsigned)((n + kThreadsMC - 1) / kThreadsMC); }

hipError_t launch_util_mc(int precision, int op, const RunMC *run, const void *fin, void *fout, double *buf,
                          int64_t nodes, hipStream_t stream)
{
    if (precision == PRECMC_FP64)
        util_mc_kernel<double><<<blocks_mc(nodes), kThreadsMC, 0, stream>>>(run, op, static_cast<const double *>(fin),
                                                                             static_cast<double *>(fout), buf);
    else
        util_mc_kernel<float><<<blocks_mc(nodes), kThreadsMC, 0, stream>>>(run, op, static_cast<const float *>(fin),
                                                                            static_cast<float *>(fout), buf);
    return hipGetLastError();
}

hipError_t launch_diag_mc(const RunMC *run, const double *buf, double cx, double cy, double r_in, double r_out,
                          double *partial, int64_t nodes, hipStream_t stream)
{
    diag_mc_kernel<<<blocks_mc(nodes), kThreadsMC, 0, stream>>>(run, buf, cx, cy, r_in, r_out, partial);
    return hipGetLastError();
}

} // namespace lbmmc
