// Host-side check of the chunked staging of the LDS tiles (ChunkPlan in
// tiles.h), built by tests/test_tile_chunks.py: over the waves of a block, every
// dword of every component of a plane is copied exactly once, from its lattice
// site, and the padding of a slot repeats the last point.  argv[1]: the turn of
// the left-over chunk.  Prints "wrong missing" for the tiles that use it.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_0901_3293_amd/csrc/tiles.h"

using hlb::wrapi;

template <class S, int NC, int E = 1>
static void check(int turn)
{
    using P = hlb::ChunkPlan<S, E>;
    const int nx = 37, ny = 21;
    long wrong = 0, missing = 0;
    for (int x0 = 0; x0 < nx; x0 += S::TX)
        for (int y0 = 0; y0 < ny; y0 += S::TY) {
            std::vector<int> times(NC * S::RS * E, 0);
            auto copy = [&](int c, int k) {
                for (int lane = 0; lane < 64; ++lane) {
                    const int e = k * 64 + lane, r = P::point(k, lane), q = e / E < S::RN ? e / E : S::RN - 1;
                    ++times[c * S::RS * E + e];
                    const int want = wrapi(x0 - 2 + q % S::RX, nx) + nx * wrapi(y0 - 2 + q / S::RX, ny);
                    wrong += hlb::TileMap<S>::staged_at(r, x0, y0, nx, ny) != want;
                }
            };
            for (int w = 0; w < P::NW; ++w) {
                for (int f = 0; f < P::FULL; ++f)
                    for (int c = 0; c < NC; ++c) copy(c, P::chunk(f, w));
                if (P::REM)
                    for (int i = 0; i < (NC + P::STEP - 1) / P::STEP; ++i)
                        if (P::left_over(i, w, turn) < NC) copy(P::left_over(i, w, turn), P::chunk(P::FULL, w));
            }
            for (int t : times) missing += t != 1;
        }
    std::printf("%ld %ld\n", wrong, missing);
}

int main(int argc, char **argv)
{
    const int turn = argc > 1 ? std::atoi(argv[1]) : 0;
    check<hlb::UpdateTile<float>, 5>(turn);
    check<hlb::UpdateTile<float>, 3>(turn);
    check<hlb::TileShape<32, 8>, 5>(turn);   // a padded slot, six waves
    check<hlb::TileShape<32, 12>, 5>(turn);  // eight waves
    check<hlb::UpdateTile<double>, 5, 2>(turn);
    check<hlb::UpdateTile<double>, 3, 2>(turn);
    return 0;
}
