// Host-side checks of the kernels that advance several steps in one launch
// (the same header functions the library uses):
//   * timed_steps: a timing of n steps of a schedule takes whole launches, at
//     least n steps and less than a launch more;
//   * tiles (every shape of the library, single and two components): the items of
//     a step are its cells and the ring around them, each once; every psi cell
//     that a collision in the grid reads was written in the same step, for the
//     neighbour that psi_coord gives; every population that a later step reads
//     was written in the step before, by the upwind node (or, across a wall, the
//     node itself, in the opposite direction); the same for the writer densities
//     of bf16 storage, from the first step on; all of them inside their LDS
//     arrays; the last step's stores cover every node of the grid once;
//   * strips: the same, with x wrapped in LDS.
// Prints "ok" and exits 0, or prints the first failure and exits 1.
#include <cstdio>
#include <vector>

#include "../paper_1306_6445_amd/csrc/lbm_kernels.hpp"
#include "../paper_1306_6445_amd/csrc/lbm_multi.hpp"

using namespace lbm;

namespace {

struct Grid {
    int nx, ny, bcx, bcy;
    int node(int x, int y) const { return psi_coord(y, ny, bcy) * nx + psi_coord(x, nx, bcx); }
};

// what one step left in an LDS array: the step that wrote a cell and the node it wrote it for
struct Cells {
    std::vector<int> step, node;
    explicit Cells(int n) : step(n, 0), node(n, -1) {}
    bool in(int i) const { return i >= 0 && i < (int)step.size(); }
    bool holds(int i, int s, int n) const { return in(i) && step[i] == s && node[i] == n; }
    bool put(int i, int s, int n)
    {
        if (!in(i)) return false;
        step[i] = s, node[i] = n;
        return true;
    }
};

#define NEED(cond, what)                                                                                          \
    do {                                                                                                          \
        if (!(cond)) {                                                                                            \
            std::printf("FAIL %s: tile %dx%d, %d steps, grid %dx%d bc %d%d, tile at (%d,%d), step %d item %d\n",  \
                        what, TX, TY, K, g.nx, g.ny, g.bcx, g.bcy, x0, y0, s, i);                                  \
            return false;                                                                                         \
        }                                                                                                         \
    } while (0)

template <int A> bool wall_of(const bool *w) { return multi_wall<A>(w); }
bool wall(int a, const bool *w)
{
    bool (*const f[9])(const bool *) = {wall_of<0>, wall_of<1>, wall_of<2>, wall_of<3>, wall_of<4>,
                                        wall_of<5>, wall_of<6>, wall_of<7>, wall_of<8>};
    return f[a](w);
}

template <int K, int TX, int TY> struct TileCheck {
    using Gm = MultiGeom<K, TX, TY>;
    const Grid g;
    const int x0, y0;
    std::vector<int> &covered;
    Cells psi, wr;
    std::vector<Cells> pop;

    TileCheck(const Grid &grid, int x, int y, std::vector<int> &c)
        : g(grid), x0(x), y0(y), covered(c), psi(Gm::PN), wr(Gm::RN), pop(9, Cells(Gm::FN))
    {
    }
    bool in_grid(int x, int y) const
    {
        return (g.bcx == BC_PERIODIC || (x >= 0 && x < g.nx)) && (g.bcy == BC_PERIODIC || (y >= 0 && y < g.ny));
    }

    template <int s> bool step()
    {
        constexpr int N = Gm::cells(s), NI = N + Gm::ring(s);
        int i = -1;
        if (s == 1) // the writer densities of the state that the launch starts from
            for (int dy = -Gm::M - 2; dy < TY + Gm::M + 2; ++dy)
                for (int dx = -Gm::M - 2; dx < TX + Gm::M + 2; ++dx)
                    NEED(wr.put(Gm::wr(dx, dy), 0, g.node(x0 + dx, y0 + dy)), "writer cell");
        std::vector<int> items((size_t)(Gm::w(s) + 2) * (Gm::h(s) + 2), 0);
        for (i = 0; i < NI; ++i) {
            int dx, dy;
            multi_item<Gm, s, K>(i, dx, dy);
            const int m = 2 * (K - s), ix = dx + m + 1, iy = dy + m + 1;
            NEED(ix >= 0 && ix < Gm::w(s) + 2 && iy >= 0 && iy < Gm::h(s) + 2, "item beyond the ring");
            NEED(items[iy * (Gm::w(s) + 2) + ix]++ == 0, "item twice");
            NEED((i < N) == (ix > 0 && ix <= Gm::w(s) && iy > 0 && iy <= Gm::h(s)), "cells first");
            const int gx = psi_coord(x0 + dx, g.nx, g.bcx), gy = psi_coord(y0 + dy, g.ny, g.bcy);
            const int cx = g.bcx == BC_WALL ? gx - x0 : dx, cy = g.bcy == BC_WALL ? gy - y0 : dy;
            const bool w[4] = {g.bcx == BC_WALL && gx == 0, g.bcx == BC_WALL && gx == g.nx - 1,
                               g.bcy == BC_WALL && gy == 0, g.bcy == BC_WALL && gy == g.ny - 1};
            for (int a = 0; a < 9; ++a) {
                const bool across = wall(a, w);
                const int from = across ? g.node(gx, gy) : g.node(gx - ex_of(a), gy - ey_of(a));
                const int writer = Gm::writer(a, Gm::wr(cx, cy), across);
                NEED(wr.holds(writer, s - 1, from), "writer density");
                if (s == 1) continue;
                const int p = Gm::pull(a, Gm::pop(cx, cy), across), slot = across ? opp_of(a) : a;
                NEED(p >= 0 && p < 9 * Gm::FN && p / Gm::FN == slot, "population array");
                NEED(pop[slot].holds(p % Gm::FN, s - 1, from), "population");
            }
            NEED(psi.put(Gm::psi(dx, dy), s, gy * g.nx + gx), "psi cell");
        }
        for (i = 0; i < (int)items.size(); ++i) NEED(items[i] == 1, "ring not covered");
        for (i = 0; i < N; ++i) {
            int dx, dy;
            multi_item<Gm, s, K>(i, dx, dy);
            const int x = x0 + dx, y = y0 + dy, node = g.node(x, y);
            for (int a = 0; a < 9 && in_grid(x, y); ++a)
                NEED(psi.holds(Gm::psi(dx, dy) + ey_of(a) * Gm::PX + ex_of(a), s, g.node(x + ex_of(a), y + ey_of(a))),
                     "psi of a neighbour");
            if (s < K) {
                // a cell beyond a wall holds no node's state
                const int tag = in_grid(x, y) ? node : -1;
                for (int a = 0; a < 9; ++a) NEED(pop[a].put(Gm::pop(dx, dy), s, tag), "population cell");
                NEED(wr.put(Gm::wr(dx, dy), s, tag), "writer cell of a collision");
            } else if (x < g.nx && y < g.ny) {
                NEED(covered[(size_t)y * g.nx + x]++ == 0, "node stored twice");
            }
        }
        if constexpr (s < K) return step<s + 1>();
        return true;
    }
};

template <int K, int TX, int TY> bool check_tiles(const Grid &g)
{
    std::vector<int> covered((size_t)g.nx * g.ny, 0);
    for (int y0 = 0; y0 < g.ny; y0 += TY)
        for (int x0 = 0; x0 < g.nx; x0 += TX)
            if (!TileCheck<K, TX, TY>(g, x0, y0, covered).template step<1>()) return false;
    for (int c : covered)
        if (c != 1) {
            std::printf("FAIL tile %dx%d, %d steps, grid %dx%d bc %d%d: node not stored\n", TX, TY, K, g.nx, g.ny,
                        g.bcx, g.bcy);
            return false;
        }
    return true;
}

template <int K, int W, int NY> struct StripCheck {
    static constexpr int TX = W, TY = NY;
    using Gm = StripGeom<K, W, NY>;
    const Grid g;
    const int x0 = 0, y0;
    std::vector<int> &covered;
    Cells psi;
    std::vector<Cells> pop;

    StripCheck(const Grid &grid, int y, std::vector<int> &c)
        : g(grid), y0(y), covered(c), psi(Gm::PN), pop(9, Cells(Gm::FN))
    {
    }

    template <int s> bool step()
    {
        constexpr int N = Gm::cells(s), NI = N + 2 * W;
        int i = -1;
        for (i = 0; i < NI; ++i) {
            const int x = i % W, dy = Gm::item_row(s, i);
            if (x >= g.nx) continue;
            const int gy = psi_coord(y0 + dy, g.ny, g.bcy);
            if (s > 1) {
                const bool w[4] = {false, false, g.bcy == BC_WALL && gy == 0, g.bcy == BC_WALL && gy == g.ny - 1};
                const int xs[3] = {x == 0 ? g.nx - 1 : x - 1, x, x == g.nx - 1 ? 0 : x + 1};
                const int row = Gm::pop(0, g.bcy == BC_WALL ? gy - y0 : dy);
                for (int a = 0; a < 9; ++a) {
                    const bool across = wall(a, w);
                    const int p = Gm::pull(a, xs, row, across), slot = across ? opp_of(a) : a;
                    NEED(p >= 0 && p < 9 * Gm::FN && p / Gm::FN == slot, "population array");
                    NEED(pop[slot].holds(p % Gm::FN, s - 1,
                                         across ? g.node(x, gy) : g.node(x - ex_of(a), gy - ey_of(a))),
                         "population");
                }
            }
            NEED(psi.put(Gm::psi(x, dy), s, g.node(x, gy)), "psi cell");
            if (x == 0) NEED(psi.put(Gm::psi(g.nx, dy), s, g.node(0, gy)), "psi copy");
            if (x == g.nx - 1) NEED(psi.put(Gm::psi(-1, dy), s, g.node(x, gy)), "psi copy");
        }
        for (i = 0; i < N; ++i) {
            const int x = i % W, dy = i / W - 2 * (K - s), y = y0 + dy;
            if (x >= g.nx) continue;
            NEED(dy == Gm::item_row(s, i), "row of a colliding item");
            const bool inside = g.bcy == BC_PERIODIC || (y >= 0 && y < g.ny);
            for (int a = 0; a < 9 && inside; ++a)
                NEED(psi.holds(Gm::psi(x, dy) + ey_of(a) * Gm::PX + ex_of(a), s, g.node(x + ex_of(a), y + ey_of(a))),
                     "psi of a neighbour");
            if (s < K) {
                for (int a = 0; a < 9; ++a) NEED(pop[a].put(Gm::pop(x, dy), s, inside ? g.node(x, y) : -1), "population cell");
            } else if (y < g.ny) {
                NEED(covered[(size_t)y * g.nx + x]++ == 0, "node stored twice");
            }
        }
        if constexpr (s < K) return step<s + 1>();
        return true;
    }
};

template <int K, int W, int TY> bool check_strips(const Grid &g)
{
    if (g.nx > W || g.bcx != BC_PERIODIC) return true;
    std::vector<int> covered((size_t)g.nx * g.ny, 0);
    for (int y0 = 0; y0 < g.ny; y0 += TY)
        if (!StripCheck<K, W, TY>(g, y0, covered).template step<1>()) return false;
    for (int c : covered)
        if (c != 1) {
            std::printf("FAIL strip %dx%d, grid %dx%d bc %d: node not stored\n", W, TY, g.nx, g.ny, g.bcy);
            return false;
        }
    return true;
}

bool check_timed_steps()
{
    for (int per : {1, 2, 4})
        for (int64_t n = 1; n <= 70; ++n) {
            const int64_t t = timed_steps(n, per);
            if (t % per != 0 || t < n || t >= n + per) {
                std::printf("FAIL timed_steps: %lld steps, %d a launch -> %lld\n", (long long)n, per, (long long)t);
                return false;
            }
        }
    return true;
}

} // namespace

int main()
{
    if (!check_timed_steps()) return 1;
    const int sizes[][2] = {{1, 1},  {2, 3},   {5, 1},   {4, 61},  {8, 51},  {7, 149}, {8, 8},   {13, 12}, {17, 33},
                            {33, 9}, {61, 25}, {64, 48}, {65, 17}, {60, 24}, {100, 5}, {121, 49}};
    int grids = 0;
    for (const auto &sz : sizes)
        for (int bc = 0; bc < 4; ++bc) {
            const Grid g{sz[0], sz[1], bc & 1, bc >> 1};
            if (!(check_tiles<4, 8, 8>(g) && check_tiles<4, 12, 12>(g) && check_tiles<4, 16, 16>(g) &&
                  check_tiles<4, 20, 20>(g) && check_tiles<2, 64, 16>(g) && check_tiles<2, 60, 24>(g) &&
                  check_tiles<2, 60, 20>(g) && check_tiles<2, 60, 12>(g) && check_tiles<2, 4, 60>(g) &&
                  check_tiles<2, 8, 60>(g) && check_tiles<2, 28, 12>(g) && check_tiles<2, 28, 20>(g) &&
                  check_tiles<2, 32, 24>(g) && check_tiles<2, 32, 16>(g) && check_tiles<2, 32, 8>(g) &&
                  check_strips<4, 4, 52>(g) && check_strips<4, 8, 50>(g)))
                return 1;
            ++grids;
        }
    std::printf("ok: %d grids\n", grids);
    return 0;
}
