// HIP kernels (gfx950) of the D3Q19 extension of the pseudopotential MRT step
// with the surface-tension source term (Li & Luo, arXiv:1306.6445, Section VI
// names 3D as future work; the 3D form follows the derivation in the design
// notes).  One step is either one launch of fused3_kernel (psi of each plane
// computed in LDS while the tile marches along z; the default) or two
// launches over the nodes of one run:
//   psi3_kernel      rho = sum_a f_a (Eq. 6) -> psi(rho) (Section II; Eq. 23)
//   collide3_kernel  psi at the 18 neighbours -> F (Eq. 7) and Q (Eq. 19) with
//                    the weights 1/6, 1/12 -> v (Eq. 6) -> m = M f -> m_eq, S
//                    (M F_Guo), C = Lambda M df((3/5) tr Q I - Q + 2 sigma
//                    |F|^2/psi^2 I) -> m* (Eq. 17) -> f* = M^-1 m* -> stored
//                    at the node in the second population buffer.
// A buffer holds the post-collision state: slot a of node y is f*_a(y) of the
// last collision.  Streaming (Eq. 4) happens as the state is read: f_a(x) =
// f*_a(x - e_a), or f*_opp(a)(x) where x - e_a lies beyond a wall (halfway
// bounce-back).  Every slot is read once per step, so reads are shifted by
// one node and writes are aligned, which streams faster on this memory system
// than aligned reads with shifted writes.
#include <hip/hip_ext.h>

#include "lbm3d_kernels.hpp"
#include "lbm_popbuf.hpp"

namespace lbm3 {

using lbm::RunDev;
using lbm::RunPar;

__host__ __device__ constexpr int c2of(int a) { return ex3(a) * ex3(a) + ey3(a) * ey3(a) + ez3(a) * ez3(a); }
// equilibrium weights (the FP32 storage's rest-state deviations) and interaction weights
__host__ __device__ constexpr double w_eq3(int a) { return c2of(a) == 0 ? 1.0 / 3.0 : (c2of(a) == 1 ? 1.0 / 18.0 : 1.0 / 36.0); }
__host__ __device__ constexpr double w_int3(int a) { return c2of(a) == 0 ? 0.0 : (c2of(a) == 1 ? 1.0 / 6.0 : 1.0 / 12.0); }

// norms of the orthogonal moment basis (rho, e, eps, jx, qx, jy, qy, jz, qz,
// 3pxx, 3pixx, pww, piww, pxy, pyz, pxz, mx, my, mz)
__host__ __device__ constexpr int mnorm(int k)
{
    return k == 0 ? 19 : k == 1 ? 2394 : k == 2 ? 252 : k <= 8 ? (k % 2 ? 10 : 40)
         : k == 9 ? 36 : k == 10 ? 72 : k == 11 ? 12 : k == 12 ? 24 : k <= 15 ? 4 : 8;
}

template <typename C> __device__ __forceinline__ C rate(const Run3 &r, int k)
{
    if constexpr (std::is_same<C, float>::value)
        return r.sf[k];
    else
        return r.s[k];
}

template <typename C> __device__ __forceinline__ C two_sigma(const Run3 &r)
{
    if constexpr (std::is_same<C, float>::value)
        return r.sig2f;
    else
        return r.sig2;
}

// Storage: FP64 populations, or FP32 deviations f_a - w_a rho_ref.
template <typename S> __device__ __forceinline__ typename std::conditional<std::is_same<S, double>::value, double, float>::type
dec(S v, int a, float ref)
{
    if constexpr (std::is_same<S, double>::value)
        return v;
    else
        return v + (float)w_eq3(a) * ref;
}
template <typename S, typename C> __device__ __forceinline__ S enc(C v, int a, float ref)
{
    if constexpr (std::is_same<S, double>::value)
        return v;
    else
        return v - (float)w_eq3(a) * ref;
}

// Eq. (6) density of 19 populations: FP64 plain sum in velocity order; FP32
// every addition made error-free by Knuth's TwoSum, the errors added once.
template <typename C> __device__ __forceinline__ C density19(const C *f)
{
    if constexpr (std::is_same<C, float>::value) {
        float s = f[0], e = 0.f;
#pragma unroll
        for (int a = 1; a < 19; ++a) {
            float ea;
            s = lbm::two_sum(s, f[a], ea);
            e += ea;
        }
        return s + e;
    } else {
        C s = f[0];
#pragma unroll
        for (int a = 1; a < 19; ++a) s += f[a];
        return s;
    }
}

__device__ __forceinline__ void coords(const Run3 &r, int64_t n, int &x, int &y, int &z)
{
    const int nx = r.r.nx, ny = r.r.ny;
    const int64_t xy = (int64_t)nx * ny;
    z = (int)(n / xy);
    const int64_t rem = n - (int64_t)z * xy;
    y = (int)(rem / nx);
    x = (int)(rem - (int64_t)y * nx);
}

__device__ __forceinline__ int64_t node_at(const Run3 &r, int x, int y, int z)
{
    return ((int64_t)z * r.r.ny + y) * r.r.nx + x;
}

// Index of the slot that holds f_a(x) of the current state (pull_slot3); the
// same map places a state given as f_a(x) into a buffer.
__device__ __forceinline__ int64_t slot3(const Run3 &r, int64_t n, const AxisNb &X, const AxisNb &Y, const AxisNb &Z,
                                         int a)
{
    return pull_slot3(n, X, Y, Z, a, r.dstride);
}

template <typename S>
__device__ __forceinline__ void gather19(const Run3 &r, const S *__restrict__ f, int64_t n, const AxisNb &X,
                                         const AxisNb &Y, const AxisNb &Z,
                                         typename std::conditional<std::is_same<S, double>::value, double, float>::type *fv)
{
    const float ref = r.r.pf.rho_ref;
#pragma unroll
    for (int a = 0; a < 19; ++a) fv[a] = dec<S>(f[slot3(r, n, X, Y, Z, a)], a, ref);
}

// The same read for a buffer of less than 4 GiB (W32): every slot's byte
// offset from the buffer's start then fits in 32 bits, so each load takes one
// offset register beside the buffer's scalar base (64-bit addresses for all
// 19 loads in flight cost the fused kernel a wave per SIMD).  Offsets wrap
// modulo 2^32 and the final offset is exact.
struct AxisNb32 {
    uint32_t m, p;
    bool wm, wp;
};
__device__ __forceinline__ AxisNb32 narrow(const AxisNb &A) { return {(uint32_t)A.m, (uint32_t)A.p, A.wm, A.wp}; }
__device__ __forceinline__ uint32_t nb_off(const AxisNb32 &A, int e) { return e > 0 ? A.p : (e < 0 ? A.m : 0u); }
__device__ __forceinline__ bool nb_wall(const AxisNb32 &A, int e) { return e > 0 ? A.wp : (e < 0 && A.wm); }

template <typename S, typename Nb>
__device__ __forceinline__ void gather19_w32(const Run3 &r, const S *__restrict__ f, uint32_t n, const Nb &X,
                                             const Nb &Y, const AxisNb32 &Z,
                                             typename std::conditional<std::is_same<S, double>::value, double, float>::type *fv)
{
    const float ref = r.r.pf.rho_ref;
    const char *base = reinterpret_cast<const char *>(f);
    const uint32_t ds = (uint32_t)r.dstride;
#pragma unroll
    for (int a = 0; a < 19; ++a) {
        const bool wall = nb_wall(X, -ex3(a)) || nb_wall(Y, -ey3(a)) || nb_wall(Z, -ez3(a));
        const uint32_t off = (uint32_t)nb_off(X, -ex3(a)) + (uint32_t)nb_off(Y, -ey3(a)) + nb_off(Z, -ez3(a));
        const uint32_t i = wall ? (uint32_t)opp3(a) * ds + n : (uint32_t)a * ds + n + off;
        fv[a] = dec<S>(*reinterpret_cast<const S *>(base + (uint32_t)(i * (uint32_t)sizeof(S))), a, ref);
    }
}

// neighbour offsets of the node n of a run
struct Nb3 {
    AxisNb X, Y, Z;
};
__device__ __forceinline__ Nb3 nb3_of(const Run3 &r, int64_t n)
{
    int x, y, z;
    coords(r, n, x, y, z);
    const int64_t sxy = (int64_t)r.r.nx * r.r.ny;
    return {axis_nb(x, r.r.nx, r.r.bc_x, 1), axis_nb(y, r.r.ny, r.r.bc_y, r.r.nx), axis_nb(z, r.nz, r.bc_z, sxy)};
}

template <typename S>
__global__ void __launch_bounds__(kThreads3) psi3_kernel(const Run3 *__restrict__ runs, const S *__restrict__ f,
                                                         void *__restrict__ psi_out, int32_t *__restrict__ status)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    const Run3 &r = runs[0];
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= r.nodes) return;
    C fv[19];
    const Nb3 nb = nb3_of(r, n);
    gather19<S>(r, f, n, nb.X, nb.Y, nb.Z, fv);
    const C rho = density19<C>(fv);
    C ps;
    const bool ok = lbm::eval_psi<C>(r.r, rho, ps);
    if (!ok) status[0] = 1;
    static_cast<C *>(psi_out)[n] = ok ? ps : C(NAN);
}

// One node's collision, shared by both schedules: psi_at(a) gives psi at
// x + e_a (a = 0: the node itself; beyond a wall, the adjacent fluid node), fv
// holds the node's 19 populations of the current state (streamed), rho their
// density19 -> fs.  The same source expressions in both kernels give the same
// bits.  Both moment transforms go through the sums and differences of
// opposite populations, which share most of their terms: about 170 additions
// and products against 400 for the rows and columns of M one by one.
template <typename C, typename PsiAt>
__device__ __forceinline__ void collide3(const RunPar<C> &k, const Run3 &r, const C *fv, C rho, const PsiAt &psi_at, C *fs)
{
    // Eq. (7) and Eq. (19) with the 3D weights 1/6 and 1/12
    C sx, sy, sz, qxx, qyy, qzz, qxy, qyz, qxz;
    const C p0 = psi_at(0);
    {
        const C w1 = C(1.0 / 6.0), w2 = C(1.0 / 12.0);
        const C p1 = psi_at(1), p2 = psi_at(2), p3 = psi_at(3), p4 = psi_at(4), p5 = psi_at(5), p6 = psi_at(6);
        const C p7 = psi_at(7), p8 = psi_at(8), p9 = psi_at(9), p10 = psi_at(10);
        const C sA = p7 + p8, sB = p9 + p10, dA = p7 - p8, dB = p9 - p10;
        const C p11 = psi_at(11), p12 = psi_at(12), p13 = psi_at(13), p14 = psi_at(14);
        const C sC = p11 + p12, sD = p13 + p14, dC = p11 - p12, dD = p13 - p14;
        const C p15 = psi_at(15), p16 = psi_at(16), p17 = psi_at(17), p18 = psi_at(18);
        const C sE = p15 + p16, sF = p17 + p18, dE = p15 - p16, dF = p17 - p18;
        sx = w1 * (p1 - p2) + w2 * ((dA + dB) + (dC + dD));
        sy = w1 * (p3 - p4) + w2 * ((dA - dB) + (dE + dF));
        sz = w1 * (p5 - p6) + w2 * ((dC - dD) + (dE - dF));
        const C xy = (sA + sB) - C(4) * p0, xz = (sC + sD) - C(4) * p0, yz = (sE + sF) - C(4) * p0;
        qxx = w1 * ((p1 + p2) - C(2) * p0) + w2 * (xy + xz);
        qyy = w1 * ((p3 + p4) - C(2) * p0) + w2 * (xy + yz);
        qzz = w1 * ((p5 + p6) - C(2) * p0) + w2 * (xz + yz);
        qxy = w2 * (sA - sB);
        qxz = w2 * (sC - sD);
        qyz = w2 * (sE - sF);
    }
    const C G = k.G;
    const C Gp = -G * p0;
    const C Fx = Gp * sx, Fy = Gp * sy, Fz = Gp * sz;
    const C F2 = G * G * (sx * sx + sy * sy + sz * sz); // |F|^2 / psi^2
    const C kq = k.kappa * G * C(0.5) * p0;
    // flux shift (3/5) tr Q I - Q + 2 sigma |F|^2/psi^2 I
    const C iso = C(0.6) * (kq * (qxx + qyy + qzz)) + two_sigma<C>(r) * F2;

    // moments from the sums and differences of opposite populations
    const C X = fv[1] + fv[2], Y = fv[3] + fv[4], Z = fv[5] + fv[6];
    const C A = fv[7] + fv[8], B = fv[9] + fv[10], Cc = fv[11] + fv[12], D = fv[13] + fv[14], E = fv[15] + fv[16],
            F = fv[17] + fv[18];
    const C dx = fv[1] - fv[2], dy = fv[3] - fv[4], dz = fv[5] - fv[6];
    const C a = fv[7] - fv[8], b = fv[9] - fv[10], c = fv[11] - fv[12], d = fv[13] - fv[14], e = fv[15] - fv[16],
            f = fv[17] - fv[18];
    const C XY = A + B, XZ = Cc + D, YZ = E + F;
    const C S1 = X + Y + Z, S2 = XY + XZ + YZ;
    const C xab = a + b, xcd = c + d, yab = a - b, yef = e + f, zcd = c - d, zef = e - f;
    const C tx = xab + xcd, ty = yab + yef, tz = zcd + zef;
    const C jx = dx + tx, jy = dy + ty, jz = dz + tz;

    // Eq. (6) velocity
    const C irho = lbm::recip<C>(rho);
    const C vx = (jx + C(0.5) * Fx) * irho, vy = (jy + C(0.5) * Fy) * irho, vz = (jz + C(0.5) * Fz) * irho;
    // P: equilibrium flux rho v v plus the flux shift; T: Guo forcing v F + F v
    const C rx = rho * vx, ry = rho * vy, rz = rho * vz;
    const C Pxx = rx * vx + (iso - kq * qxx), Pyy = ry * vy + (iso - kq * qyy), Pzz = rz * vz + (iso - kq * qzz);
    const C Pxy = rx * vy - kq * qxy, Pyz = ry * vz - kq * qyz, Pxz = rx * vz - kq * qxz;
    const C Txx = C(2) * (vx * Fx), Tyy = C(2) * (vy * Fy), Tzz = C(2) * (vz * Fz);
    const C Txy = vx * Fy + vy * Fx, Tyz = vy * Fz + vz * Fy, Txz = vx * Fz + vz * Fx;
    const C trP = Pxx + Pyy + Pzz, trT = Txx + Tyy + Tzz;

    // Eq. (17): m* = m + s (m_eq + C - m) + (1 - s/2) S, scaled by 1 / norm.
    // Conserved moments: rho* = rho, and with the Eq. (6) velocity
    // j* = j - s_j (j - rho v) + (1 - s_j/2) F = j + F for any s_j; through
    // div_const (in FP32 the product with a rounded 1/19 or 1/10 would bias the
    // mass and momentum by an ulp every step; the residual correction removes it)
    auto relax = [&](int q, C m, C target, C force) {
        const C s = rate<C>(r, q);
        return (m + s * (target - m) + (C(1) - C(0.5) * s) * force) * C(1.0 / mnorm(q));
    };
    const C me = relax(1, C(-30) * fv[0] - C(11) * S1 + C(8) * S2, C(-11) * rho + C(19) * trP, C(19) * trT);
    const C mp = relax(2, C(12) * fv[0] - C(4) * S1 + S2, C(3) * rho - C(5.5) * trP, C(-5.5) * trT);
    const C gx = relax(4, tx - C(4) * dx, C(-2.0 / 3.0) * rx, C(-2.0 / 3.0) * Fx);
    const C gy = relax(6, ty - C(4) * dy, C(-2.0 / 3.0) * ry, C(-2.0 / 3.0) * Fy);
    const C gz = relax(8, tz - C(4) * dz, C(-2.0 / 3.0) * rz, C(-2.0 / 3.0) * Fz);
    const C ax2 = C(2) * X - (Y + Z), dg2 = (XY + XZ) - C(2) * YZ;
    const C P3 = C(3) * Pxx - trP, T3 = C(3) * Txx - trT;
    const C m9 = relax(9, ax2 + dg2, P3, T3);
    const C m10 = relax(10, dg2 - C(2) * ax2, C(-0.5) * P3, C(-0.5) * T3);
    const C axw = Y - Z, dgw = XY - XZ, Pw = Pyy - Pzz, Tw = Tyy - Tzz;
    const C m11 = relax(11, axw + dgw, Pw, Tw);
    const C m12 = relax(12, dgw - C(2) * axw, C(-0.5) * Pw, C(-0.5) * Tw);
    const C mxy = relax(13, A - B, Pxy, Txy), myz = relax(14, E - F, Pyz, Tyz), mxz = relax(15, Cc - D, Pxz, Txz);
    auto decay = [&](int q, C m) { return (m - rate<C>(r, q) * m) * C(1.0 / mnorm(q)); };
    const C mx = decay(16, xab - xcd), my = decay(17, yef - yab), mz = decay(18, zcd - zef);
    const C m0 = lbm::div_const<C>(rho, 19.0);
    const C hx = lbm::div_const<C>(jx + Fx, 10.0), hy = lbm::div_const<C>(jy + Fy, 10.0),
            hz = lbm::div_const<C>(jz + Fz, 10.0);

    // f* = M^T of the scaled moments, opposite populations together
    fs[0] = m0 - C(30) * me + C(12) * mp;
    const C ax = m0 - C(11) * me - C(4) * mp, dg = m0 + C(8) * me + mp;
    auto pair = [](C even, C odd, C &plus, C &minus) {
        plus = even + odd;
        minus = even - odd;
    };
    const C px = m9 - C(2) * m10, pw = m11 - C(2) * m12;
    pair(ax + C(2) * px, hx - C(4) * gx, fs[1], fs[2]);
    pair((ax - px) + pw, hy - C(4) * gy, fs[3], fs[4]);
    pair((ax - px) - pw, hz - C(4) * gz, fs[5], fs[6]);
    const C dp = m9 + m10, dw = m11 + m12, ux = hx + gx, uy = hy + gy, uz = hz + gz;
    const C exy = (dg + dp) + dw, exz = (dg + dp) - dw, eyz = dg - C(2) * dp;
    const C xp = ux + mx, xm = ux - mx, yp = uy + my, ym = uy - my, zp = uz + mz, zm = uz - mz;
    pair(exy + mxy, xp + ym, fs[7], fs[8]);
    pair(exy - mxy, xp - ym, fs[9], fs[10]);
    pair(exz + mxz, xm + zp, fs[11], fs[12]);
    pair(exz - mxz, xm - zp, fs[13], fs[14]);
    pair(eyz + myz, yp + zm, fs[15], fs[16]);
    pair(eyz - myz, yp - zm, fs[17], fs[18]);
}

// The collide pass runs over tiles of 2^txs x (256 >> txs) nodes in x-y, one
// z-plane each; the 1D work index decomposes with workgroup-uniform integer
// arithmetic, so no thread divides.  Workgroups reach the XCDs round-robin;
// work_index gives each XCD a contiguous range of tiles, so the neighbours
// whose gathers share cache lines (x), and whose psi rows and planes a tile
// reads (y, z), run under the same L2.
template <typename S>
__global__ void __launch_bounds__(kThreads3) collide3_kernel(const Run3 *__restrict__ runs, const S *__restrict__ fin,
                                                             S *__restrict__ fout, const void *__restrict__ psi_in,
                                                             int txs)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    const Run3 &r = runs[0];
    const int nx = r.r.nx, ny = r.r.ny, nz = r.nz, bcx = r.r.bc_x, bcy = r.r.bc_y, bcz = r.bc_z;
    int x, y, z;
    if (!collide3_node((unsigned)lbm::work_index(1), threadIdx.x, nx, ny, nz, txs, x, y, z)) return;
    const int64_t sxy = (int64_t)nx * ny;
    const int64_t n = (int64_t)z * sxy + (int64_t)y * nx + x;
    const AxisNb X = axis_nb(x, nx, bcx, 1), Y = axis_nb(y, ny, bcy, nx), Z = axis_nb(z, nz, bcz, sxy);
    const C *psi = static_cast<const C *>(psi_in);
    C fv[19];
    gather19<S>(r, fin, n, X, Y, Z, fv);
    C fs[19];
    collide3<C>(r.r.template par<C>(), r, fv, density19<C>(fv), [&](int a) {
        return psi[n + nb_off(X, ex3(a)) + nb_off(Y, ey3(a)) + nb_off(Z, ez3(a))];
    }, fs);
    // f* stays at the node; the next read streams it (Eq. 4)
    const float ref = r.r.pf.rho_ref;
#pragma unroll
    for (int a = 0; a < 19; ++a) fout[(int64_t)a * r.dstride + n] = enc<S, C>(fs[a], a, ref);
}

// The fused step: one launch, psi computed where it is needed.  A workgroup
// owns an x-y tile of TX x TY nodes and marches along z through a chunk of
// planes.  psi of the plane ahead (the tile and a one-node ring around it; the
// ring and any tile column beyond the grid take the wrapped or clamped node)
// goes into one of four rotating LDS planes; after one barrier the tile's
// nodes of the current plane collide with the psi of planes z - 1, z, z + 1
// and store into the other buffer.  Each node's populations are gathered once
// (streamed from planes z, z + 1, z + 2 of the source), for its psi, and wait
// in the thread's own LDS column for their collision one plane later (FP32: all in
// registers took 128 of them; FP64: see fused3_park).  The ring's populations are
// re-read from cache.  Four slots let one barrier per plane suffice: the slot a
// plane's psi goes into was last read two planes earlier, before the previous
// barrier.  Out of place, so every workgroup reads only the unmodified source
// buffer.
// What bounds it: a plane is a chain of load latency, density, barrier and
// collision, so each thread loads the populations of the plane after next
// before it collides (160^3 FP32 171 -> 154 us a step; the ring's loads ahead as
// well cost registers, 220 us), and the 38 shifted or aligned streams, which
// move 5.0 TB/s of counted traffic at 256^3 against 5.14 of a probe without
// arithmetic.  160^3 FP32 304 -> 147 us with the chunk of its default schedule,
// 256^3 619 -> 549, 96^3 FP64 517 -> 60.
//
// How a tile's populations are addressed (MODE), the same slots in each:
//   kFlat   no wall within reach and each buffer below 4 GiB: a buffer
//           descriptor, one 32-bit offset per (ex, ey) and a scalar one per
//           direction and plane, so a load takes no vector address arithmetic;
//   kWall32 walls, below 4 GiB; kWide 64-bit addresses.
constexpr int kFlat = 0, kWall32 = 1, kWide = 2;

// Directions whose waiting populations sit in LDS, beside the four psi planes in
// the 160 KB of a CU; the others wait in registers.  All 19 where they fit, but
//  - 12 in FP64 with 512 threads and 32-bit offsets, whose 256 registers hold the
//    other 7: with all in registers the kernel spilled 104 bytes a lane, with all
//    in LDS it is slower (160^3 266 us a step spilling, 268 with 12 or 8, 276 with
//    19; 256^3 1024, 1026, 1055).  With 64-bit addresses 19 are faster (320 x 320 x
//    328: 2325 us, 2476 with 12, 3418 spilling);
//  - 15 in FP64 with 1,024 threads, all that fit (128 registers: what is left over
//    spills, and no loads ahead: 160^3 521 us, 1588 with all in registers).
template <typename C> constexpr int fused3_park(int TX, int TY, bool w32)
{
    const int fit = (163840 / (int)sizeof(C) - 4 * (TX + 2) * (TY + 2)) / (TX * TY);
    if (sizeof(C) == 8 && TX * TY == 512 && w32) return 12;
    return fit < 19 ? fit : 19;
}

template <typename S, int TX, int TY, int MODE, bool NTS>
__device__ __forceinline__ bool fused3_tile(const Run3 &r, const S *__restrict__ fin, S *__restrict__ fout,
                                            const Fused3Thread &q,
                                            typename std::conditional<std::is_same<S, double>::value, double, float>::type *lps,
                                            typename std::conditional<std::is_same<S, double>::value, double, float>::type *park)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    constexpr int PX = TX + 2, PLANE = PX * (TY + 2), NT = TX * TY;
    constexpr int PARK = fused3_park<C>(TX, TY, MODE != kWide);
    // loads ahead of the collision where the registers hold them
    constexpr bool AHEAD = sizeof(C) == 4 || NT <= 512;
    constexpr uint32_t sz = sizeof(S);
    const int nx = r.r.nx, ny = r.r.ny, nz = r.nz, bcx = r.r.bc_x, bcy = r.r.bc_y, bcz = r.bc_z;
    const RunPar<C> k = r.r.template par<C>();
    const float ref = r.r.pf.rho_ref;
    const int64_t sxy = (int64_t)nx * ny;
    const uint32_t ds = (uint32_t)r.dstride * sz, plane = (uint32_t)sxy * sz;
    const lbm::PopBuf<S> in(fin), out(fout);

    // populations of the column (cx, cy) on plane z (wrapped or clamped)
    auto gather = [&](int z, int cx, int cy, int64_t col, C *fv) {
        if constexpr (MODE == kFlat) {
            const uint32_t xo[3] = {(uint32_t)(cx == 0 ? nx - 1 : cx - 1) * sz, (uint32_t)cx * sz,
                                    (uint32_t)(cx == nx - 1 ? 0 : cx + 1) * sz};
            const uint32_t row = (uint32_t)nx * sz;
            const uint32_t yo[3] = {(uint32_t)(cy == 0 ? ny - 1 : cy - 1) * row, (uint32_t)cy * row,
                                    (uint32_t)(cy == ny - 1 ? 0 : cy + 1) * row};
            const uint32_t zo[3] = {(uint32_t)(z == 0 ? nz - 1 : z - 1) * plane, (uint32_t)z * plane,
                                    (uint32_t)(z == nz - 1 ? 0 : z + 1) * plane};
#pragma unroll
            for (int a = 0; a < 19; ++a)
                fv[a] = dec<S>(in.load(xo[1 - ex3(a)] + yo[1 - ey3(a)], a * ds + zo[1 - ez3(a)]), a, ref);
        } else {
            const AxisNb X = axis_nb(cx, nx, bcx, 1), Y = axis_nb(cy, ny, bcy, nx), Z = axis_nb(z, nz, bcz, sxy);
            if constexpr (MODE == kWall32)
                gather19_w32<S>(r, fin, (uint32_t)(z * sxy + col), narrow(X), narrow(Y), narrow(Z), fv);
            else
                gather19<S>(r, fin, z * sxy + col, X, Y, Z, fv);
        }
    };
    bool bad = false;
    auto put_psi = [&](int zl, int cell, const C *fv) {
        const C rho = density19<C>(fv);
        C ps;
        const bool ok = lbm::eval_psi<C>(k, r.r.eos_kind, rho, ps);
        lps[(zl & 3) * PLANE + cell] = ok ? ps : C(NAN);
        bad |= !ok;
        return rho;
    };
    const int tid = (int)threadIdx.x;
    C kept[PARK < 19 ? 19 - PARK : 1];
    C rc = C(0); // density of the waiting populations
    C fv[19]; // populations of the next plane, loaded ahead of the collision
    if (AHEAD) gather(lbm::psi_coord(q.z0 - 1, nz, bcz), q.cx, q.cy, q.col, fv);
    for (int zl = q.z0 - 1; zl <= q.z1; ++zl) {
        // psi of plane zl, tile and ring
        if (q.ring) {
            C fr[19];
            gather(lbm::psi_coord(zl, nz, bcz), q.rcx, q.rcy, q.rcol, fr);
            put_psi(zl, q.rcell, fr);
        }
        if (!AHEAD) gather(lbm::psi_coord(zl, nz, bcz), q.cx, q.cy, q.col, fv);
        const C rho = put_psi(zl, q.cell, fv);
        // the populations of plane zl - 1 out, those of zl in
        C fc[19];
#pragma unroll
        for (int a = 0; a < 19; ++a) {
            if (a < PARK) {
                fc[a] = park[a * NT + tid];
                park[a * NT + tid] = fv[a];
            } else {
                fc[a] = kept[a - PARK];
                kept[a - PARK] = fv[a];
            }
        }
        const C rcc = rc;
        rc = rho;
        __syncthreads();
        if (AHEAD && zl < q.z1) gather(lbm::psi_coord(zl + 1, nz, bcz), q.cx, q.cy, q.col, fv);
        const int z = zl - 1;
        if (z < q.z0 || !q.active) continue;
        C fs[19];
        collide3<C>(k, r, fc, rcc, [&](int a) {
            return lps[((z + ez3(a)) & 3) * PLANE + q.cell + ey3(a) * PX + ex3(a)];
        }, fs);
        // f* stays at the node; the next read streams it (Eq. 4)
        if constexpr (MODE == kWide) {
            const int64_t n = (int64_t)z * sxy + (int64_t)q.y * nx + q.x;
#pragma unroll
            for (int a = 0; a < 19; ++a) fout[(int64_t)a * r.dstride + n] = enc<S, C>(fs[a], a, ref);
        } else {
#pragma unroll
            for (int a = 0; a < 19; ++a)
                out.template store<NTS>((uint32_t)(q.y * nx + q.x) * sz, a * ds + (uint32_t)z * plane, enc<S, C>(fs[a], a, ref));
        }
    }
    return bad;
}

template <typename S, int TX, int TY, bool W32, bool NTS>
__global__ void __launch_bounds__(TX * TY) fused3_kernel(const Run3 *__restrict__ runs, const S *__restrict__ fin,
                                                         S *__restrict__ fout, int32_t *__restrict__ status, int zc)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    constexpr int PLANE = (TX + 2) * (TY + 2), NT = TX * TY;
    static_assert(PLANE - NT <= NT, "one ring node per thread at most");
    __shared__ C lps[4 * PLANE], park[fused3_park<C>(TX, TY, W32) * NT];
    const Run3 &r = runs[0];
    const int nx = r.r.nx, ny = r.r.ny, nz = r.nz;
    const Fused3Thread q = fused3_thread((unsigned)lbm::work_index(1), threadIdx.x, nx, ny, nz, r.r.bc_x, r.r.bc_y, zc, TX, TY);
    bool bad;
    if constexpr (W32) {
        // walls within two nodes of the workgroup's tile and planes
        const int x0 = q.x - (int)threadIdx.x % TX, y0 = q.y - (int)threadIdx.x / TX;
        const bool flat = (r.r.bc_x == lbm::BC_PERIODIC || (x0 >= 2 && x0 + TX + 2 <= nx)) &&
                          (r.r.bc_y == lbm::BC_PERIODIC || (y0 >= 2 && y0 + TY + 2 <= ny)) &&
                          (r.bc_z == lbm::BC_PERIODIC || (q.z0 >= 2 && q.z1 + 2 <= nz));
        if (flat)
            bad = fused3_tile<S, TX, TY, kFlat, NTS>(r, fin, fout, q, lps, park);
        else
            bad = fused3_tile<S, TX, TY, kWall32, NTS>(r, fin, fout, q, lps, park);
    } else {
        bad = fused3_tile<S, TX, TY, kWide, NTS>(r, fin, fout, q, lps, park);
    }
    if (bad) status[0] = 1;
}

// ------------------------------------------------------------- utilities

template <typename S>
__global__ void util3_kernel(const Run3 *__restrict__ runs, int op, const S *__restrict__ fin, S *__restrict__ fout,
                             const void *__restrict__ psi_in, double *__restrict__ buf)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    const Run3 &r = runs[0];
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t N = r.nodes;
    if (n >= N) return;
    const float ref = r.r.pf.rho_ref;
    const Nb3 nb = nb3_of(r, n);
    if (op == 0) {
        C fv[19];
        gather19<S>(r, fin, n, nb.X, nb.Y, nb.Z, fv);
#pragma unroll
        for (int a = 0; a < 19; ++a) buf[a * N + n] = (double)fv[a];
    } else if (op == 2) {
        // f_a(x) into the slot it is read from (each slot written once)
#pragma unroll
        for (int a = 0; a < 19; ++a) fout[slot3(r, n, nb.X, nb.Y, nb.Z, a)] = enc<S, C>((C)buf[a * N + n], a, ref);
    } else if (op == 3) {
        const double rho = buf[n], v[3] = {buf[N + n], buf[2 * N + n], buf[3 * N + n]};
        const double v2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
#pragma unroll
        for (int a = 0; a < 19; ++a) {
            const double eu = ex3(a) * v[0] + ey3(a) * v[1] + ez3(a) * v[2];
            const double fe = w_eq3(a) * rho * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * v2);
            fout[slot3(r, n, nb.X, nb.Y, nb.Z, a)] = enc<S, C>((C)fe, a, ref);
        }
    } else {
        // density and Eq. (6) velocity in FP64 from psi of the same state
        const C *psi = static_cast<const C *>(psi_in);
        C fv[19];
        gather19<S>(r, fin, n, nb.X, nb.Y, nb.Z, fv);
        double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < 19; ++a) {
            rho += (double)fv[a];
            j[0] += ex3(a) * (double)fv[a];
            j[1] += ey3(a) * (double)fv[a];
            j[2] += ez3(a) * (double)fv[a];
        }
        int x, y, z;
        coords(r, n, x, y, z);
        double s[3] = {0.0, 0.0, 0.0};
        for (int a = 1; a < 19; ++a) {
            const int gx = lbm::psi_coord(x + ex3(a), r.r.nx, r.r.bc_x), gy = lbm::psi_coord(y + ey3(a), r.r.ny, r.r.bc_y),
                      gz = lbm::psi_coord(z + ez3(a), r.nz, r.bc_z);
            const double pa = (double)psi[node_at(r, gx, gy, gz)];
            s[0] += w_int3(a) * pa * ex3(a);
            s[1] += w_int3(a) * pa * ey3(a);
            s[2] += w_int3(a) * pa * ez3(a);
        }
        const double p0 = (double)psi[n], G = r.r.pd.G;
        buf[n] = rho;
        for (int i = 0; i < 3; ++i) buf[(i + 1) * N + n] = (j[i] - 0.5 * G * p0 * s[i]) / rho;
    }
}

template <typename S>
__global__ void __launch_bounds__(kThreads3) diag3_kernel(const Run3 *__restrict__ runs, const S *__restrict__ f,
                                                          const void *__restrict__ psi_in, int dims, double cx,
                                                          double cy, double cz, double r_in, double r_out,
                                                          double *__restrict__ partial)
{
    using C = typename std::conditional<std::is_same<S, double>::value, double, float>::type;
    __shared__ double red[8][kThreads3];
    const Run3 &r = runs[0];
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int tid = threadIdx.x;
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (n < r.nodes) {
        const C *psi = static_cast<const C *>(psi_in);
        C fv[19];
        const Nb3 nb = nb3_of(r, n);
        gather19<S>(r, f, n, nb.X, nb.Y, nb.Z, fv);
        double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < 19; ++a) {
            rho += (double)fv[a];
            j[0] += ex3(a) * (double)fv[a];
            j[1] += ey3(a) * (double)fv[a];
            j[2] += ez3(a) * (double)fv[a];
        }
        int x, y, z;
        coords(r, n, x, y, z);
        double s[3] = {0.0, 0.0, 0.0};
        for (int a = 1; a < 19; ++a) {
            const int gx = lbm::psi_coord(x + ex3(a), r.r.nx, r.r.bc_x), gy = lbm::psi_coord(y + ey3(a), r.r.ny, r.r.bc_y),
                      gz = lbm::psi_coord(z + ez3(a), r.nz, r.bc_z);
            const double pa = (double)psi[node_at(r, gx, gy, gz)];
            s[0] += w_int3(a) * pa * ex3(a);
            s[1] += w_int3(a) * pa * ey3(a);
            s[2] += w_int3(a) * pa * ez3(a);
        }
        const double p0 = (double)psi[n], G = r.r.pd.G;
        double sp2 = 0.0;
        for (int i = 0; i < 3; ++i) {
            const double u = (j[i] - 0.5 * G * p0 * s[i]) / rho;
            sp2 += u * u;
        }
        // minimum-image distance on periodic axes; dims 2: a cylinder along z
        double dx = x - cx, dy = y - cy, dz = dims == 3 ? z - cz : 0.0;
        if (r.r.bc_x == lbm::BC_PERIODIC) dx -= r.r.nx * rint(dx / r.r.nx);
        if (r.r.bc_y == lbm::BC_PERIODIC) dy -= r.r.ny * rint(dy / r.r.ny);
        if (dims == 3 && r.bc_z == lbm::BC_PERIODIC) dz -= r.nz * rint(dz / r.nz);
        const double dist = sqrt(dx * dx + dy * dy + dz * dz);
        const double p = lbm::eval_pressure(r.r, rho);
        v[0] = rho;
        if (dist <= r_in) {
            v[1] = rho;
            v[2] = 1.0;
            v[5] = p;
        }
        if (dist >= r_out) {
            v[3] = rho;
            v[4] = 1.0;
            v[6] = p;
        }
        const double sp = sqrt(sp2);
        v[7] = sp == sp ? sp : INFINITY;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) red[q][tid] = v[q];
    __syncthreads();
    for (int s = kThreads3 / 2; s > 0; s >>= 1) {
        if (tid < s) {
#pragma unroll
            for (int q = 0; q < 7; ++q) red[q][tid] += red[q][tid + s];
            red[7][tid] = fmax(red[7][tid], red[7][tid + s]);
        }
        __syncthreads();
    }
    if (tid < 8) partial[(int64_t)blockIdx.x * 8 + tid] = red[tid][0];
}

// ------------------------------------------------------------- launchers

static unsigned blocks3(int64_t n) { return (unsigned)((n + kThreads3 - 1) / kThreads3); }

template <typename S, int TX, int TY> hipError_t fused3_t(const Step3Args &a)
{
    const dim3 grid(fused3_blocks(a.nx, a.ny, a.nz, TX, TY, a.zchunk)), block(TX * TY);
    auto go = [&](auto kernel) {
        hipExtLaunchKernelGGL(kernel, grid, block, 0, a.stream, a.ev_col0, a.ev_col1, 0, a.run,
                              static_cast<const S *>(a.fin), static_cast<S *>(a.fout), a.status, a.zchunk);
    };
    if (!a.w32)
        go(fused3_kernel<S, TX, TY, false, false>);
    else if (a.beyond_cache)
        go(fused3_kernel<S, TX, TY, true, true>);
    else
        go(fused3_kernel<S, TX, TY, true, false>);
    return hipGetLastError();
}

template <typename S> hipError_t fused3_shape(const Step3Args &a)
{
    switch (a.tile_x * 100 + a.tile_y) {
    case 3208: return fused3_t<S, 32, 8>(a);
    case 3216: return fused3_t<S, 32, 16>(a);
    case 6404: return fused3_t<S, 64, 4>(a);
    case 6416: return fused3_t<S, 64, 16>(a);
    default: return fused3_t<S, 64, 8>(a);
    }
}

template <typename S> hipError_t step3_t(const Step3Args &a)
{
    if (a.fused) return fused3_shape<S>(a);
    const unsigned nb = blocks3(a.nodes);
    hipExtLaunchKernelGGL(psi3_kernel<S>, dim3(nb), dim3(kThreads3), 0, a.stream, a.ev_psi0, a.ev_psi1, 0, a.run,
                          static_cast<const S *>(a.fin), a.psi, a.status);
    hipExtLaunchKernelGGL(collide3_kernel<S>, dim3(collide3_blocks(a.nx, a.ny, a.nz)), dim3(kThreads3), 0,
                          a.stream, a.ev_col0, a.ev_col1, 0, a.run, static_cast<const S *>(a.fin),
                          static_cast<S *>(a.fout), (const void *)a.psi, collide3_tile_shift(a.nx));
    return hipGetLastError();
}

hipError_t launch_step3(int precision, const Step3Args &a)
{
    return precision == PREC3_FP64 ? step3_t<double>(a) : step3_t<float>(a);
}

hipError_t launch_psi3(int precision, const Run3 *run, const void *f, void *psi, int32_t *status, int64_t nodes,
                       hipStream_t stream)
{
    if (precision == PREC3_FP64)
        psi3_kernel<double><<<blocks3(nodes), kThreads3, 0, stream>>>(run, static_cast<const double *>(f), psi, status);
    else
        psi3_kernel<float><<<blocks3(nodes), kThreads3, 0, stream>>>(run, static_cast<const float *>(f), psi, status);
    return hipGetLastError();
}

template <typename S>
hipError_t util3_t(int op, const Run3 *run, const void *fin, void *fout, const void *psi, double *buf, int64_t nodes,
                   hipStream_t stream)
{
    util3_kernel<S><<<blocks3(nodes), kThreads3, 0, stream>>>(run, op, static_cast<const S *>(fin),
                                                               static_cast<S *>(fout), psi, buf);
    return hipGetLastError();
}

hipError_t launch_util3(int precision, int op, const Run3 *run, const void *fin, void *fout, const void *psi,
                        double *buf, int64_t nodes, hipStream_t stream)
{
    return precision == PREC3_FP64 ? util3_t<double>(op, run, fin, fout, psi, buf, nodes, stream)
                                   : util3_t<float>(op, run, fin, fout, psi, buf, nodes, stream);
}

template <typename S>
hipError_t diag3_t(const Run3 *run, const void *f, const void *psi, int dims, double cx, double cy, double cz,
                   double r_in, double r_out, double *partial, int64_t nodes, hipStream_t stream)
{
    diag3_kernel<S><<<blocks3(nodes), kThreads3, 0, stream>>>(run, static_cast<const S *>(f), psi, dims, cx, cy, cz,
                                                               r_in, r_out, partial);
    return hipGetLastError();
}

hipError_t launch_diag3(int precision, const Run3 *run, const void *f, const void *psi, int dims, double cx,
                        double cy, double cz, double r_in, double r_out, double *partial, int64_t nodes,
                        hipStream_t stream)
{
    return precision == PREC3_FP64 ? diag3_t<double>(run, f, psi, dims, cx, cy, cz, r_in, r_out, partial, nodes, stream)
                                   : diag3_t<float>(run, f, psi, dims, cx, cy, cz, r_in, r_out, partial, nodes, stream);
}

} // namespace lbm3
