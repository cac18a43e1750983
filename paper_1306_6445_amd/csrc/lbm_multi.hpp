// Tiles of the kernels that advance several 2D steps in one launch.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_device.hpp"

namespace lbm {

// Geometry of a tile of TX x TY nodes advanced K steps: step s (1..K) collides
// the tile and a margin of 2 (K - s) nodes around it, for which it needs psi
// one node further out.
template <int K, int TX, int TY> struct MultiGeom {
    static constexpr int M = 2 * (K - 1);                       // margin of the first step
    static constexpr int FX = TX + 2 * M, FY = TY + 2 * M, FN = FX * FY; // LDS populations
    static constexpr int PX = FX + 2, PN = PX * (FY + 2);       // LDS psi
    static constexpr int RX = FX + 4, RN = RX * (FY + 4);       // LDS writer densities (bf16 storage)
    static constexpr int w(int s) { return TX + 4 * (K - s); }
    static constexpr int h(int s) { return TY + 4 * (K - s); }
    static constexpr int cells(int s) { return w(s) * h(s); }
    static constexpr int ring(int s) { return 2 * (w(s) + 2) + 2 * h(s); }
    // LDS cell of the node at (dx, dy) from the tile's origin: populations, psi, writer
    // densities (where the kernels write pop and psi out, the call compiles to more instructions)
    __host__ __device__ static constexpr int pop(int dx, int dy) { return (dy + M) * FX + dx + M; }
    __host__ __device__ static constexpr int psi(int dx, int dy) { return (dy + M + 1) * PX + dx + M + 1; }
    __host__ __device__ static constexpr int wr(int dx, int dy) { return (dy + M + 2) * RX + dx + M + 2; }
    // LDS slot of f_a streamed to the node of population cell c: slot a of x - e_a, or across a wall its own opp(a)
    __host__ __device__ static constexpr int pull(int a, int c, bool wall)
    {
        return wall ? opp_of(a) * FN + c : a * FN + c - (ey_of(a) * FX + ex_of(a));
    }
    // cell of the writer of f_a at the node of writer cell c
    __host__ __device__ static constexpr int writer(int a, int c, bool wall)
    {
        return wall ? c : c - (ey_of(a) * RX + ex_of(a));
    }
};

// Whether f_A reaches across a wall a node that touches those of w: below and above
// in x, below and above in y.
template <int A> __host__ __device__ __forceinline__ bool multi_wall(const bool *w)
{
    constexpr int ex = ex_of(A), ey = ey_of(A);
    return (ex > 0 && w[0]) || (ex < 0 && w[1]) || (ey > 0 && w[2]) || (ey < 0 && w[3]);
}

// Position, relative to the tile's origin, of item k of step s: first the
// colliding cells row by row, then the one-node ring around them (top row,
// bottom row, left and right columns).
template <typename Gm, int s, int K> __host__ __device__ __forceinline__ void multi_item(int k, int &dx, int &dy)
{
    constexpr int W = Gm::w(s), H = Gm::h(s), N = Gm::cells(s), m = 2 * (K - s);
    if (k < N) {
        const int ly = (unsigned)k / (unsigned)W;
        dx = k - ly * W - m;
        dy = ly - m;
    } else {
        const int q = k - N;
        const bool rows = q < 2 * (W + 2);
        const bool second = rows ? q >= W + 2 : (q & 1);
        const int c = rows ? (second ? q - (W + 2) : q) : (q - 2 * (W + 2)) >> 1;
        dx = rows ? c - 1 - m : (second ? W - m : -1 - m);
        dy = rows ? (second ? H - m : -1 - m) : c - m;
    }
}

// Geometry of a strip: the whole width of a grid of at most W nodes along a
// periodic x by TY rows, x wrapped in LDS, a margin along y only.
template <int K, int W, int TY> struct StripGeom {
    static constexpr int M = 2 * (K - 1), FN = W * (TY + 2 * M); // LDS populations, W columns a row
    static constexpr int PX = W + 2, PN = PX * (TY + 2 * M + 2); // LDS psi, a copied column either side
    static constexpr int cells(int s) { return W * (TY + 4 * (K - s)); }
    __host__ __device__ static constexpr int pop(int x, int dy) { return (dy + M) * W + x; }
    __host__ __device__ static constexpr int psi(int x, int dy) { return (dy + M + 1) * PX + x + 1; }
    // row of item i of step s: the rows that collide, then one above and one below that need only psi
    __host__ __device__ static constexpr int item_row(int s, int i)
    {
        return i < cells(s) ? i / W - 2 * (K - s) : (i < cells(s) + W ? -1 - 2 * (K - s) : TY + 2 * (K - s));
    }
    // LDS slot of f_a streamed to column xs[1] of the row that starts at cell r; xs: the columns before, at and after
    __host__ __device__ static constexpr int pull(int a, const int *xs, int r, bool wall)
    {
        return wall ? opp_of(a) * FN + r + xs[1] : a * FN + r - ey_of(a) * W + xs[1 - ex_of(a)];
    }
};

constexpr int kMGeneral = 0, kMPeriodic = 1, kMInner = 2;

} // namespace lbm
