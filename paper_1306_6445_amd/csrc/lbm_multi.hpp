// Tiles of the kernels that advance several 2D steps in one launch.
#pragma once

#include <hip/hip_runtime.h>

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
};

// Position, relative to the tile's origin, of item k of step s: first the
// colliding cells row by row, then the one-node ring around them (top row,
// bottom row, left and right columns).
template <typename Gm, int s, int K> __device__ __forceinline__ void multi_item(int k, int &dx, int &dy)
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

constexpr int kMGeneral = 0, kMPeriodic = 1, kMInner = 2;

} // namespace lbm
