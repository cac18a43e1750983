// Several D2Q9 steps in one launch (every storage, single-range force):
// multi_kernel reads the populations of an even step count, advances its tile
// K steps with the intermediate states in LDS and writes the state K steps
// later, in the same layout, to the other buffer.
//
// Why: one step per launch reads and writes every population of the grid each
// step (72 B per node and step in FP32), which bounded the grids that do not
// fit a cache, and costs a launch and a chain of dependent loads, which
// bounded the small ones.  Step s of the K collides the tile and a margin of
// 2 (K - s) nodes, for which it needs psi one node further out, so the margin's
// work is done again by the neighbouring tiles: for K = 2 1.16 collisions and 1.33
// densities per node and step with 64 x 16 tiles, 1.12 and 1.25 with 60 x 24.  HBM
// traffic halves (FP32, by the counters: 72 B per node and 2 steps on 40 grids of
// 256^2, 83 on 4096 x 2048) and the kernel is bound by vector instruction issue: 404
// and 371 a node and step there.
// The intermediate state passes through LDS in its storage form (FP32
// deviations; bf16 with its writer densities and rounding bits), so that K steps
// in one launch and K launches give the same bits.
//
// Measured against one step per launch (us per step): 4096 x 2048 FP32 142 ->
// 88, FP64 261 -> 158; 40 x 256^2 FP32 32.7 -> 25.1, FP64 87 -> 57; 64 uneven
// drops FP32 128 -> 77; 2048 x 1024 with walls FP32 27.8 -> 21; 100^2 FP64 6.0 ->
// 2.2; 256 grids of 4 x 256 FP32 38 -> 3.75 (strips); 40 x 256^2 bf16 40.9 -> 32.1, 64
// uneven drops bf16 125 -> 93.
#include <hip/hip_ext.h>

#include "lbm_device.hpp"
#include "lbm_kernels.hpp"
#include "lbm_multi.hpp"
#include "lbm_node.hpp"
#include "lbm_popbuf.hpp"

namespace lbm {

template <typename S, int K, int TX, int TY, int NT, int MODE>
struct MultiTile {
    using C = typename Store<S>::C;
    using Gm = MultiGeom<K, TX, TY>;
    const RunPar<C> k;
    const int eos, nx, ny, ld, bcx, bcy, x0, y0;
    const uint32_t ds; // bytes from one direction's array to the next
    const PopBuf<S> in, out;
    C *psi;
    S *pop;
    // bf16 storage: the writer densities that decode the current state (of the
    // previous step's nodes; a colliding node replaces its own), the array of
    // the last step's densities, the first step's rounding seed, the run's
    // first node (for the rounding hash)
    float *wr;
    float *rlast;
    uint32_t seed;
    int64_t n_off;
    bool bad = false;

    template <int A> __device__ __forceinline__ C decode(S v, C base) const { return Store<S>::template load<A>(&v, 0, base); }
    // hb: the node's rounding bits, advanced once per population
    template <int A> __device__ __forceinline__ S encode(C v, C base, uint32_t &hb) const
    {
        if constexpr (kWriterRef<S>) {
            hb = hb * 747796405u + 2891336453u;
            return Store<S>::template encode_sr_hw<A>(v, base, hb);
        } else {
            S r;
            Store<S>::template store<A>(&r, 0, v, base);
            return r;
        }
    }
    // base density of f_a of the item's node: its writer's (x - e_a, or x across a wall), or the run's constant
    template <int A> __device__ __forceinline__ C base_of(int wc, bool wall) const
    {
        if constexpr (kWriterRef<S>)
            return C(wr[Gm::writer(A, wc, wall)]);
        else
            return k.rho_ref;
    }
    // the node an item stands for: wrapped on periodic axes (global), clamped across walls
    __device__ __forceinline__ int wrap_x(int x) const { return MODE == kMInner ? x : psi_coord(x, nx, MODE == kMPeriodic ? BC_PERIODIC : bcx); }
    __device__ __forceinline__ int wrap_y(int y) const { return MODE == kMInner ? y : psi_coord(y, ny, MODE == kMPeriodic ? BC_PERIODIC : bcy); }

    struct LoadG {
        const MultiTile &t;
        uint32_t off;
        int wc;
        bool w[4];
        C *f;
        template <int A> __device__ __forceinline__ void operator()()
        {
            const bool wall = MODE == kMGeneral && kWriterRef<S> && multi_wall<A>(w);
            f[A] = t.template decode<A>(t.in.load(off, A * t.ds), t.template base_of<A>(wc, wall));
        }
    };
    // f_a(x) of an intermediate state: f*_a(x - e_a), or f*_opp(a)(x) across a wall
    struct LoadL {
        const MultiTile &t;
        int cell, wc; // of the item's node
        bool w[4];
        C *f;
        template <int A> __device__ __forceinline__ void operator()()
        {
            const bool wall = MODE == kMGeneral && multi_wall<A>(w);
            f[A] = t.template decode<A>(t.pop[Gm::pull(A, cell, wall)], t.template base_of<A>(wc, wall));
        }
    };
    struct StoreL {
        const MultiTile &t;
        int cell;
        const C *f;
        C base;
        uint32_t hb;
        template <int A> __device__ __forceinline__ void operator()()
        {
            t.pop[A * Gm::FN + cell] = t.template encode<A>(f[A], base, hb);
        }
    };
    // f*_a(x) to slot a of x + e_a, or slot opp(a) of x across a wall (the even-state layout)
    struct StoreG {
        const MultiTile &t;
        uint32_t xo[3], yo[3]; // byte offsets of x - 1, x, x + 1 and of rows y - 1, y, y + 1
        bool wxm, wxp, wym, wyp;
        const C *f;
        C base;
        uint32_t hb;
        template <int A> __device__ __forceinline__ void operator()()
        {
            constexpr int ex = ex_of(A), ey = ey_of(A);
            const S v = t.template encode<A>(f[A], base, hb);
            if constexpr (MODE == kMInner) {
                t.out.store(xo[1], A * t.ds + (uint32_t)((ey * t.ld + ex) * (int)sizeof(S)), v);
            } else if constexpr (MODE == kMPeriodic || A == 0) {
                t.out.store(xo[1 + ex] + yo[1 + ey], A * t.ds, v);
            } else {
                const bool wall = (ex > 0 && wxp) || (ex < 0 && wxm) || (ey > 0 && wyp) || (ey < 0 && wym);
                t.out.store(wall ? opp_of(A) * t.ds + xo[1] + yo[1] : A * t.ds + xo[1 + ex] + yo[1 + ey], 0, v);
            }
        }
    };

    template <int s> __device__ __forceinline__ void load(int dx, int dy, C *f) const
    {
        const int gx = wrap_x(x0 + dx), gy = wrap_y(y0 + dy);
        // LDS cell: unwrapped on a periodic axis, the clamped node's across a wall
        int cx = dx, cy = dy;
        bool w[4] = {false, false, false, false};
        if constexpr (MODE == kMGeneral) {
            if (bcx == BC_WALL) cx = gx - x0, w[0] = gx == 0, w[1] = gx == nx - 1;
            if (bcy == BC_WALL) cy = gy - y0, w[2] = gy == 0, w[3] = gy == ny - 1;
        }
        const int wc = Gm::wr(cx, cy);
        if constexpr (s == 1) {
            LoadG op{*this, (uint32_t)(gy * ld + gx) * (uint32_t)sizeof(S), wc, {w[0], w[1], w[2], w[3]}, f};
            for9(op);
        } else {
            LoadL op{*this, (cy + Gm::M) * Gm::FX + cx + Gm::M, wc, {w[0], w[1], w[2], w[3]}, f};
            for9(op);
        }
    }

    template <int s> __device__ __forceinline__ C put_psi(int dx, int dy, const C *f)
    {
        C ps, rho;
        bad |= !node_psi<C>(k, eos, f, ps, rho);
        psi[Gm::psi(dx, dy)] = ps;
        return rho;
    }

    template <int s> __device__ __forceinline__ void step(int tid)
    {
        constexpr int N = Gm::cells(s), NI = N + Gm::ring(s), R = (N + NT - 1) / NT;
        C fv[R][9], rho[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT;
            if (i < NI) {
                int dx, dy;
                multi_item<Gm, s, K>(i, dx, dy);
                load<s>(dx, dy, fv[j]);
                rho[j] = put_psi<s>(dx, dy, fv[j]);
            }
        }
        for (int i = tid + R * NT; i < NI; i += NT) {
            int dx, dy;
            multi_item<Gm, s, K>(i, dx, dy);
            C fr[9];
            load<s>(dx, dy, fr);
            put_psi<s>(dx, dy, fr);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT;
            if (i < N) {
                const int ly = (unsigned)i / (unsigned)Gm::w(s), lx = i - ly * Gm::w(s);
                const int dx = lx - 2 * (K - s), dy = ly - 2 * (K - s);
                C fs[9];
                collide_node<C>(k, fv[j], rho[j], psi + (dy + Gm::M + 1) * Gm::PX + dx + Gm::M + 1, Gm::PX, fs);
                // bf16 storage: this node's density is the base of what it writes, rounded stochastically
                C base = k.rho_ref;
                uint32_t hb = 0;
                int64_t gi = 0;
                if constexpr (kWriterRef<S>) {
                    base = rho[j];
                    gi = n_off + (int64_t)wrap_y(y0 + dy) * ld + wrap_x(x0 + dx);
                    hb = fmix32((uint32_t)gi ^ fmix32(seed + (s - 1)));
                }
                if constexpr (s < K) {
                    if constexpr (kWriterRef<S>) wr[Gm::wr(dx, dy)] = (float)rho[j];
                    StoreL op{*this, (dy + Gm::M) * Gm::FX + dx + Gm::M, fs, base, hb};
                    for9(op);
                } else {
                    const int x = x0 + dx, y = y0 + dy;
                    if (MODE == kMInner || (x < nx && y < ny)) {
                        constexpr uint32_t z = sizeof(S);
                        if constexpr (kWriterRef<S>) rlast[gi] = (float)rho[j];
                        StoreG op{*this, {}, {}, false, false, false, false, fs, base, hb};
                        if constexpr (MODE == kMInner) {
                            op.xo[1] = (uint32_t)(y * ld + x) * z;
                        } else {
                            const Nbr n = neighbours(x, y, nx, ny, MODE == kMPeriodic ? BC_PERIODIC : bcx,
                                                     MODE == kMPeriodic ? BC_PERIODIC : bcy);
                            op.xo[0] = n.xm * z, op.xo[1] = x * z, op.xo[2] = n.xp * z;
                            op.yo[0] = n.ym * ld * z, op.yo[1] = y * ld * z, op.yo[2] = n.yp * ld * z;
                            op.wxm = n.wxm, op.wxp = n.wxp, op.wym = n.wym, op.wyp = n.wyp;
                        }
                        for9(op);
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

// LDS of a tile: psi, the intermediate populations, the writer densities.
template <typename S, int K, int TX, int TY> struct MultiLds {
    using Gm = MultiGeom<K, TX, TY>;
    typename Store<S>::C psi[Gm::PN];
    float wr[kWriterRef<S> ? Gm::RN : 1];
    S pop[9 * Gm::FN];
};

template <typename S, int K, int TX, int TY, int NT, int MODE>
__device__ __forceinline__ bool multi_tile(const RunDev &r, const Tile &t, const S *src, S *dst,
                                           MultiLds<S, K, TX, TY> &lds, float *rlast, uint32_t seed)
{
    MultiTile<S, K, TX, TY, NT, MODE> m{r.template par<typename Store<S>::C>(), r.eos_kind, r.nx, r.ny, r.pitch, r.bc_x,
                                       r.bc_y, t.x0, t.y0, (uint32_t)r.dstride * (uint32_t)sizeof(S), PopBuf<S>(src),
                                       PopBuf<S>(dst), lds.psi, lds.pop, lds.wr, rlast, seed, r.n_off};
    m.template step<1>((int)threadIdx.x);
    return m.bad;
}

// Grid: one workgroup per tile of the list, or of the one run (ntx tiles to a
// row).  bf16 storage: rprev holds the densities of the last step, rlast
// receives those of this launch's last step; seeds holds the rounding seeds
// of the last even and odd step, seeds_out receives this launch's (other
// arrays, because every workgroup reads the old ones).
template <typename S, int K, int TX, int TY, int NT>
__global__ void __launch_bounds__(NT) multi_kernel(const RunDev *__restrict__ runs, const Tile *__restrict__ tiles, int ntx,
                                              const S *__restrict__ src, S *__restrict__ dst,
                                              int32_t *__restrict__ status, int xcd, const float *__restrict__ rprev,
                                              float *__restrict__ rlast, const uint32_t *__restrict__ seeds,
                                              uint32_t *__restrict__ seeds_out)
{
    static_assert(K % 2 == 0, "the state returns to the layout of an even step count");
    using Gm = MultiGeom<K, TX, TY>;
    __shared__ __align__(16) MultiLds<S, K, TX, TY> lds;
    const int wi = work_index(xcd);
    // one run: the tile follows from the work index (no dependent load of the list)
    const Tile t = ntx > 0 ? Tile{0, wi % ntx * TX, wi / ntx * TY, 0} : tiles[wi];
    const RunDev &r = runs[t.run];
    uint32_t seed = 0;
    if constexpr (kWriterRef<S>) {
        seed = seeds[1] + 1u;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            seeds_out[0] = seed + (K - 2);
            seeds_out[1] = seed + (K - 1);
        }
        const float *rp = rprev + r.n_off;
        for (int i = threadIdx.x; i < Gm::RN; i += NT) {
            const int ly = (unsigned)i / (unsigned)Gm::RX, lx = i - ly * Gm::RX;
            const int gx = psi_coord(t.x0 + lx - (Gm::M + 2), r.nx, r.bc_x);
            const int gy = psi_coord(t.y0 + ly - (Gm::M + 2), r.ny, r.bc_y);
            lds.wr[i] = rp[(int64_t)gy * r.pitch + gx];
        }
        __syncthreads();
    }
    constexpr int E = Gm::M + 2; // reach of the first step's loads and of the last step's stores
    const bool inner = t.x0 - E >= 0 && t.x0 + TX + E <= r.nx && t.y0 - E >= 0 && t.y0 + TY + E <= r.ny;
    const S *in = src + r.f_off;
    S *out = dst + r.f_off;
    bool bad;
    if (inner)
        bad = multi_tile<S, K, TX, TY, NT, kMInner>(r, t, in, out, lds, rlast, seed);
    else if (r.bc_x == BC_PERIODIC && r.bc_y == BC_PERIODIC)
        bad = multi_tile<S, K, TX, TY, NT, kMPeriodic>(r, t, in, out, lds, rlast, seed);
    else
        bad = multi_tile<S, K, TX, TY, NT, kMGeneral>(r, t, in, out, lds, rlast, seed);
    if (bad) status[t.run] = 1;
}

// Grids of at most W nodes along a periodic x (flat slabs).  A tile of the
// kernel above repeats such a grid in its margins: 12 columns of collisions for
// 4 nodes.  Here a tile is the whole width by TY rows, x wraps in LDS, and only
// the rows have a margin.
//  - LDS: the populations W columns a row, psi with a copied column either side.
//  - An item is a node of a row (W = 4 or 8: shifts; columns past nx idle), then
//    the 2 W nodes of the rows above and below that need only psi.
// 256 grids of 4 x 256, us a step: FP32 3.75 against 6.2 with 4 x 60 tiles of the
// kernel above (which collides 1.6 cells a node and step; here 1.13), FP64 5.8
// against 9.6; 16 of them 1.9 / 2.4.  Vector issue bounds many grids, the chain of
// four steps a few.
template <typename S, int K, int W, int TY, int NT> struct StripTile {
    using C = typename Store<S>::C;
    using Gm = StripGeom<K, W, TY>;
    const RunPar<C> k;
    const int eos, nx, ny, ld, bcy, y0;
    const uint32_t ds; // bytes from one direction's array to the next
    const PopBuf<S> in, out;
    C *psi;
    S *pop;
    bool bad = false;

    template <int A> __device__ __forceinline__ C decode(S v) const { return Store<S>::template load<A>(&v, 0, k.rho_ref); }

    struct LoadG {
        const StripTile &t;
        uint32_t off;
        C *f;
        template <int A> __device__ __forceinline__ void operator()() { f[A] = t.template decode<A>(t.in.load(off, A * t.ds)); }
    };
    // f_a(x) of an intermediate state: f*_a(x - e_a), or f*_opp(a)(x) across a wall
    struct LoadL {
        const StripTile &t;
        int row, xs[3]; // first cell of the node's row; x - 1, x, x + 1
        bool wym, wyp;
        C *f;
        template <int A> __device__ __forceinline__ void operator()()
        {
            const bool wall = (ey_of(A) > 0 && wym) || (ey_of(A) < 0 && wyp);
            f[A] = t.template decode<A>(t.pop[Gm::pull(A, xs, row, wall)]);
        }
    };
    struct StoreL {
        const StripTile &t;
        int cell;
        const C *f;
        template <int A> __device__ __forceinline__ void operator()()
        {
            Store<S>::template store<A>(t.pop, A * Gm::FN + cell, f[A], t.k.rho_ref);
        }
    };
    // f*_a(x) to slot a of x + e_a, or slot opp(a) of x across a wall (the even-state layout)
    struct StoreG {
        const StripTile &t;
        uint32_t xo[3], yo[3]; // byte offsets of x - 1, x, x + 1 and of rows y - 1, y, y + 1
        bool wym, wyp;
        const C *f;
        template <int A> __device__ __forceinline__ void operator()()
        {
            constexpr int ex = ex_of(A), ey = ey_of(A);
            S v;
            Store<S>::template store<A>(&v, 0, f[A], t.k.rho_ref);
            const bool wall = (ey > 0 && wyp) || (ey < 0 && wym);
            t.out.store(wall ? opp_of(A) * t.ds + xo[1] + yo[1] : A * t.ds + xo[1 + ex] + yo[1 + ey], 0, v);
        }
    };

    template <int s> __device__ __forceinline__ C density(int x, int dy, C *f)
    {
        const int gy = psi_coord(y0 + dy, ny, bcy);
        if constexpr (s == 1) {
            LoadG op{*this, (uint32_t)(gy * ld + x) * (uint32_t)sizeof(S), f};
            for9(op);
        } else {
            // LDS row: unwrapped on a periodic axis, the clamped node's across a wall
            const bool wall = bcy == BC_WALL;
            LoadL op{*this, Gm::pop(0, wall ? gy - y0 : dy), {x == 0 ? nx - 1 : x - 1, x, x == nx - 1 ? 0 : x + 1},
                     wall && gy == 0, wall && gy == ny - 1, f};
            for9(op);
        }
        C ps, rho;
        bad |= !node_psi<C>(k, eos, f, ps, rho);
        psi[Gm::psi(x, dy)] = ps;
        if (x == 0) psi[Gm::psi(nx, dy)] = ps;
        if (x == nx - 1) psi[Gm::psi(-1, dy)] = ps;
        return rho;
    }

    template <int s> __device__ __forceinline__ void step(int tid)
    {
        constexpr int N = Gm::cells(s), NI = N + 2 * W, R = (N + NT - 1) / NT;
        C fv[R][9], rho[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT, x = i % W;
            // past the cells come the ring rows; an item of them needs no populations later
            if (i < NI && x < nx) rho[j] = density<s>(x, Gm::item_row(s, i), fv[j]);
        }
        for (int i = tid + R * NT; i < NI; i += NT) {
            C fr[9];
            if (i % W < nx) density<s>(i % W, Gm::item_row(s, i), fr);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * NT, x = i % W, dy = i / W - 2 * (K - s);
            if (i < N && x < nx) {
                C fs[9];
                collide_node<C>(k, fv[j], rho[j], psi + Gm::psi(x, dy), Gm::PX, fs);
                if constexpr (s < K) {
                    StoreL op{*this, Gm::pop(x, dy), fs};
                    for9(op);
                } else if (y0 + dy < ny) {
                    constexpr uint32_t z = sizeof(S);
                    const Nbr n = neighbours(x, y0 + dy, nx, ny, BC_PERIODIC, bcy);
                    StoreG op{*this, {n.xm * z, x * z, n.xp * z}, {n.ym * ld * z, (y0 + dy) * ld * z, n.yp * ld * z},
                              n.wym, n.wyp, fs};
                    for9(op);
                }
            }
        }
        if constexpr (s < K) {
            __syncthreads();
            step<s + 1>(tid);
        }
    }
};

template <typename S, int K, int W, int TY, int NT>
__global__ void __launch_bounds__(NT) strip_kernel(const RunDev *__restrict__ runs, const Tile *__restrict__ tiles, int ntx,
                                              const S *__restrict__ src, S *__restrict__ dst,
                                              int32_t *__restrict__ status, int xcd)
{
    static_assert(K % 2 == 0, "the state returns to the layout of an even step count");
    static_assert(!kWriterRef<S>, "FP64 and FP32 storage");
    using C = typename Store<S>::C;
    using T = StripTile<S, K, W, TY, NT>;
    __shared__ C psi[T::Gm::PN];
    __shared__ S pop[9 * T::Gm::FN];
    const int wi = work_index(xcd);
    const Tile t = ntx > 0 ? Tile{0, 0, wi * TY, 0} : tiles[wi];
    const RunDev &r = runs[t.run];
    T m{r.template par<C>(), r.eos_kind, r.nx, r.ny, r.pitch, r.bc_y, t.y0, (uint32_t)r.dstride * (uint32_t)sizeof(S),
        PopBuf<S>(src + r.f_off), PopBuf<S>(dst + r.f_off), psi, pop};
    m.template step<1>((int)threadIdx.x);
    if (m.bad) status[t.run] = 1;
}

} // namespace lbm

// ------------------------------------------------------------ launchers
namespace lbm {

namespace {

template <typename S, int K, int TX, int TY, int NT> hipError_t launch_multi_t(const StepArgs &a)
{
    hipExtLaunchKernelGGL((multi_kernel<S, K, TX, TY, NT>), dim3(a.nmtiles), dim3(NT), 0, a.stream, a.ev_start, a.ev_stop,
                          0, a.runs, a.mtiles, a.mntx, static_cast<const S *>(a.f), static_cast<S *>(a.f_alt), a.status,
                          a.xcd, a.r1, a.r0, a.seed, a.seed_alt);
    return hipGetLastError();
}

template <typename S, int K, int W, int TY, int NT> hipError_t launch_strip_t(const StepArgs &a)
{
    hipExtLaunchKernelGGL((strip_kernel<S, K, W, TY, NT>), dim3(a.nmtiles), dim3(NT), 0, a.stream, a.ev_start, a.ev_stop,
                          0, a.runs, a.mtiles, a.mntx, static_cast<const S *>(a.f), static_cast<S *>(a.f_alt), a.status,
                          a.xcd);
    return hipGetLastError();
}

struct Variant {
    MultiShape shape;
    // vector instructions of a tile, about 93 per density and 200 per collision, times what it loses otherwise
    int64_t work;
    // small tiles of several steps: taken when the work list has no more of them than this
    int64_t max_tiles;
    hipError_t (*launch)(const StepArgs &);
    bool strip; // grids of at most tile-width nodes along a periodic x; taken where every run is one
};

template <typename S, int K, int TX, int TY, int NT> constexpr Variant make_variant(int64_t max_tiles, int percent = 100)
{
    using Gm = MultiGeom<K, TX, TY>;
    int64_t work = 0;
    for (int s = 1; s <= K; ++s) work += 93 * (Gm::cells(s) + Gm::ring(s)) + 200 * Gm::cells(s);
    return {{K, TX, TY}, work * percent / 100, max_tiles, launch_multi_t<S, K, TX, TY, NT>, false};
}

template <typename S, int K, int W, int TY, int NT> constexpr Variant make_strip()
{
    return {{K, W, TY}, 0, INT64_MAX, launch_strip_t<S, K, W, TY, NT>, true};
}

// The variants of one precision: strips, then the latency-bound ones (max_tiles >
// 0).  The threads of a strip hold the first step's cells and its two ring rows in
// one round (256 threads for 4 x 52: 2.0 us instead of 1.9 for one 4 x 256 grid;
// K = 2 4.6 instead of 3.75 for 256; 4 x 64 and 8 x 64 lose 10-25% on heights
// that they do not divide).
// Threads of a tile are a multiple of 256 (four waves, one per SIMD: 576 ran 20%
// slower than 512), and the first step's cells fill them in one or two rounds,
// those of 60 x 24 (1,792 on 768 threads) in two and a third.
//  - K = 4 tiles for few nodes, where a step is the launch and one chain of
//    latencies: the smaller the tile the shorter the chain, as long as each
//    tile has a CU of its own, 256 of them (FP32, us a step: 180^2 2.23 with 12 x
//    12 against 2.7 with 529 tiles of 8 x 8, 256^2 2.44 with 16 x 16 against 2.74
//    with 20 x 20, 300^2 2.85 with 20 x 20 against 3.23; bf16 180^2 2.75 / 3.3,
//    256^2 2.98 / 3.34), then two to a CU (350^2 3.3 with 16 x 16 against 3.8;
//    FP64 256^2 3.8 with 12 x 12 against 3.87 with 28 x 12 and K = 2);
//  - otherwise the shape with the least work, counting whole tiles: 60 x 24 has
//    the smallest margins that leave two workgroups a CU (72 KB of LDS; 4096 x
//    2048 87.7 us against 89.0 with 60 x 20, 2048 x 1024 20.4 against 21.4; 60 x
//    44, one workgroup a CU, 113.6), 60 x 20 and 64 x 16 fit some heights and widths
//    better (40 x 100^2 7.3 against 8.2, 40 x 256^2 25.5 against 27.3; 1280 x 1024
//    15.0 against 15.4 at equal work, hence the charge of 1%), 4 x 60 and 8 x 60
//    grids a few nodes wide that no strip takes (256 of 4 x 256: 5.9 us against 12
//    with 16 x 16 tiles and 32 with 60 x 20).
//  - FP64 takes 32 x 24: 1008 cells in two rounds of 512 threads, rows that start
//    on 256 bytes, two workgroups in the 160 KB (4096 x 2048 158 us against 181 with
//    28 x 20 and 176 with 32 x 16, more than their work explains: the charges of 8
//    and 5%; 768 threads 232), and those two where they fit better (40 x 100^2 12.3
//    against 13.6).
const Variant kF32[] = {
    make_strip<float, 4, 4, 52, 320>(), make_strip<float, 4, 8, 50, 512>(),
    make_variant<float, 4, 8, 8, 512>(256),  make_variant<float, 4, 12, 12, 768>(256),
    make_variant<float, 4, 16, 16, 1024>(256), make_variant<float, 4, 20, 20, 1024>(256),
    make_variant<float, 4, 16, 16, 1024>(512), make_variant<float, 4, 20, 20, 1024>(512),
    make_variant<float, 2, 64, 16, 768>(0),  make_variant<float, 2, 60, 24, 768>(0, 101),
    make_variant<float, 2, 60, 20, 768>(0),
    make_variant<float, 2, 4, 60, 512>(0),   make_variant<float, 2, 8, 60, 768>(0),
};
const Variant kF64[] = {
    make_strip<double, 4, 4, 52, 320>(), make_strip<double, 4, 8, 50, 512>(),
    make_variant<double, 4, 8, 8, 512>(256), make_variant<double, 4, 12, 12, 768>(512),
    make_variant<double, 2, 28, 12, 512>(768), make_variant<double, 2, 32, 24, 512>(0),
    make_variant<double, 2, 32, 16, 512>(0, 105), make_variant<double, 2, 28, 20, 768>(0, 108),
    make_variant<double, 2, 4, 60, 512>(0),
};

// bf16 storage spends its time on decoding and rounding (480 instructions a node
// and step): 512 threads for 64 x 16 tiles measured 32.1 us on 40 x 256^2 drops
// against 32.5 with 768 and 34.9 with 64 x 12 tiles.
const Variant kBf16[] = {
    make_variant<bf16_t, 4, 8, 8, 512>(256),   make_variant<bf16_t, 4, 12, 12, 768>(256),
    make_variant<bf16_t, 4, 16, 16, 1024>(256), make_variant<bf16_t, 4, 20, 20, 1024>(256),
    make_variant<bf16_t, 2, 28, 12, 512>(768), make_variant<bf16_t, 2, 64, 16, 512>(0),
    make_variant<bf16_t, 2, 60, 12, 512>(0),   make_variant<bf16_t, 2, 4, 60, 512>(0),
};

const Variant *variant(int precision, int v)
{
    if (precision == PREC_FP32) return v >= 0 && v < (int)(sizeof(kF32) / sizeof(kF32[0])) ? &kF32[v] : nullptr;
    if (precision == PREC_FP64) return v >= 0 && v < (int)(sizeof(kF64) / sizeof(kF64[0])) ? &kF64[v] : nullptr;
    if (precision == PREC_BF16) return v >= 0 && v < (int)(sizeof(kBf16) / sizeof(kBf16[0])) ? &kBf16[v] : nullptr;
    return nullptr;
}

} // namespace

bool multi_shape(int precision, int v, MultiShape &s)
{
    const Variant *p = variant(precision, v);
    if (p) s = p->shape;
    return p != nullptr;
}

// Vector instructions of a single step with tiles of tx x (rows ty) nodes (93 per
// density, 200 per collision, as above): waves beyond the grid's last row or
// column do no work, the ring is whole.
static int64_t single_work(const RunDev &r, int tx, int ty, int rows)
{
    const int wide = tx < 64 ? tx : 64, high = ty * rows;
    const int64_t tiles = multi_tiles({1, tx, high}, r.nx, r.ny);
    return (int64_t)((r.nx + wide - 1) / wide * wide) * r.ny * (93 + 200) + tiles * 93 * (2 * (tx + 2) + 2 * high);
}

// Besides the shapes' own rules, single steps stay where the rows of tiles beyond
// flat grids cost more than the launches save: when the tiles outnumber the
// resident workgroups (three a CU in bf16, two otherwise), several steps a launch
// are taken up to 1.65 times the work of as many single steps.  Measured, us a
// step, single against several: at 1.5 times the work 200 grids of 64 x 34 FP32 9.5
// / 8.9, FP64 15.4 / 14.3; at 1.6 100 of 400 x 8 bf16 10.9 / 8.5; at 1.7 200000 x 8
// bf16 29.3 / 29.5; at 2.2 200000 x 8 FP32 23.7 / 27.4, FP64 39.9 / 49.0, 100 of 400 x
// 8 8.3 / 8.3 and 13.0 / 13.9; at 4 1000000 x 4 FP32 78 / 113.  With fewer tiles the
// chain of a launch counts, not the work (at 2.2 20000 x 8 FP32 6.3 / 5.7, at 1.7
// 40000 x 8 bf16 10.8 / 8.2).
int pick_multi(int precision, const RunDev *runs, int nruns, int tx, int ty, int rows)
{
    int best = -1;
    int64_t least = 0, single = 0, launched = 0;
    for (int i = 0; i < nruns; ++i) single += single_work(runs[i], tx, ty, rows);
    for (int v = 0; const Variant *p = variant(precision, v); ++v) {
        int64_t tiles = 0;
        bool fits = true;
        for (int i = 0; i < nruns; ++i) {
            tiles += multi_tiles(p->shape, runs[i].nx, runs[i].ny);
            fits &= !p->strip || (runs[i].nx <= p->shape.tx && runs[i].bc_x == BC_PERIODIC);
        }
        if (!fits) continue;
        if (p->max_tiles > 0) {
            if (tiles <= p->max_tiles) return v;
        } else if (best < 0 || tiles * p->work < least) {
            best = v;
            least = tiles * p->work;
            launched = tiles;
        }
    }
    const int64_t resident = precision == PREC_BF16 ? 768 : 512;
    return best >= 0 && launched > resident && 100 * least > 165 * variant(precision, best)->shape.steps * single ? -1 : best;
}

hipError_t launch_multi(int precision, int v, const StepArgs &a)
{
    const Variant *p = variant(precision, v);
    return p && a.f_alt && (a.mntx > 0 || a.mtiles) ? p->launch(a) : hipErrorInvalidValue;
}

} // namespace lbm
