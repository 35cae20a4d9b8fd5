// Host-side check of the LDS planes that are copied straight from global memory,
// built by tests/test_tile_planes.py.  Stages one plane of every component the way
// the kernels do (ChunkPlan and TileMap::staged_at, dword by dword, into NaN) and
// reads what their stencils read: the evaluation point of every thread and its four
// in-plane neighbours.  Prints for each tile in use "wrong" (dwords of another site
// or component, or never staged), "cover" (points of the halo-1 plane not evaluated
// exactly once, tile sites not their thread's own).  argv[1] plants a mistake in the
// staging: 1 the left-over chunk of wave 0 is not copied, 2 a lane's neighbour is.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_0901_3293_amd/csrc/tiles.h"

using hlb::wrapi;

template <class S, int NC, int E>
static void check(int turn, int drop)
{
    using P = hlb::ChunkPlan<S, E>;
    using M = hlb::TileMap<S>;
    // lattices and tile origins: whole tiles, tiles hanging over by some sites or rows, lattices smaller than a tile
    const int cases[][4] = {{128, 130, 64, 125}, {150, 94, 128, 90}, {126, 129, 64, 125}, {200, 60, 192, 55},
                            {13, 7, 0, 0},       {4, 4, 0, 0},       {64, 4, 0, 0},       {129, 35, 96, 32}};
    long wrong = 0, cover = 0;
    for (const auto &cs : cases) {
        const int nx = cs[0], ny = cs[1], x0 = cs[2], y0 = cs[3];
        std::vector<long> slot(NC * S::RS * E, -1);  // (component, site, dword) that was copied, or none
        auto copy = [&](int w, int c, int k) {
            if (drop == 1 && w == 0 && P::LEFT && k >= P::FULL * P::NW) return;
            for (int lane = 0; lane < 64; ++lane) {
                const int r = P::point(k, drop == 2 && lane ? lane - 1 : lane), e = k * 64 + lane;
                slot[c * S::RS * E + e] = (long(c) * nx * ny + M::staged_at(r, x0, y0, nx, ny)) * E + lane % E;
            }
        };
        for (int w = 0; w < P::NW; ++w) {
            for (int f = 0; f < P::FULL; ++f)
                for (int c = 0; c < NC; ++c) copy(w, c, P::chunk(f, w));
            for (int i = 0; P::LEFT && i < (NC + P::STEP - 1) / P::STEP; ++i)
                if (P::left_over(i, w, turn) < NC) copy(w, P::left_over(i, w, turn), P::chunk(P::FULL, w));
        }
        std::vector<int> evaluated(S::PN, 0);
        for (int t = 0; t < S::NB; ++t) {
            int pc, rc;
            if (!M::point(t, pc, rc)) continue;
            ++evaluated[pc];
            if (t < S::NT) {
                int opc, orc;
                M::own(t, opc, orc);
                cover += opc != pc || orc != rc;
            }
            for (int c = 0; c < NC; ++c)
                for (int d : {0, 1, -1, S::RX, -S::RX}) {
                    const int o = rc + d, x = wrapi(x0 - 2 + o % S::RX, nx), y = wrapi(y0 - 2 + o / S::RX, ny);
                    for (int e = 0; e < E; ++e)
                        wrong += slot[(c * S::RS + o) * E + e] != (long(c) * nx * ny + x + nx * y) * E + e;
                }
        }
        for (int v : evaluated) cover += v != 1;
    }
    std::printf("%ld %ld\n", wrong, cover);
}

int main(int argc, char **argv)
{
    const int drop = argc > 1 ? std::atoi(argv[1]) : 0;
    check<hlb::WideTile<float>, 5, 1>(0, drop);  // fused stress and LB
    check<hlb::WideTile<double>, 5, 2>(0, drop);
    check<hlb::KernelTile<float>, 5, 1>(0, drop);
    check<hlb::KernelTile<double>, 5, 2>(0, drop);
    check<hlb::UpdateTile<float>, 5, 1>(0, drop);  // Q update: Q, and u with the left-over chunks turned
    check<hlb::UpdateTile<float>, 3, 1>(hlb::ChunkPlan<hlb::UpdateTile<float>, 1>::STEP - 1, drop);
    check<hlb::UpdateTile<double>, 5, 2>(0, drop);
    check<hlb::UpdateTile<double>, 3, 2>(hlb::ChunkPlan<hlb::UpdateTile<double>, 2>::STEP - 1, drop);
    return 0;
}
