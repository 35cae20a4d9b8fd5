// Host build of the rules of tiles.h that choose a form of a step by the size of
// the lattice, for tests/test_tile_rules.py.  argv: rule (with its
// argument), precision (32, 64), CUs, then nx ny nz of each lattice; prints one value a lattice.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../paper_0901_3293_amd/csrc/tiles.h"

template <typename T>
static int rule(const char *name, int nx, int ny, int nz, int cus)
{
    if (!std::strcmp(name, "pass_chunk_force")) return hlb::pass_chunk<T>(nx, ny, nz, cus, false);
    if (!std::strcmp(name, "pass_chunk_split")) return hlb::pass_chunk<T>(nx, ny, nz, cus, true);
    // chunk of the Q update, the whole-stress kernel, the wide fused one with `argument` blocks a CU
    if (!std::strncmp(name, "fill_update_", 12))
        return hlb::fill_chunk<hlb::UpdateTile<T>>(nx, ny, nz, (long long)cus * std::atoi(name + 12));
    if (!std::strncmp(name, "fill_stress_", 12))
        return hlb::fill_chunk<hlb::KernelTile<T>>(nx, ny, nz, (long long)cus * std::atoi(name + 12));
    if (!std::strncmp(name, "fill_wide_", 10))
        return hlb::fill_chunk<hlb::WideTile<T>>(nx, ny, nz, (long long)cus * std::atoi(name + 10));
    if (!std::strncmp(name, "wide_", 5)) return hlb::wide_tiles<T>(nx, ny, nz, cus, std::atoi(name + 5));
    return -1;
}

int main(int argc, char **argv)
{
    for (int i = 4; i + 2 < argc; i += 3) {
        const int nx = std::atoi(argv[i]), ny = std::atoi(argv[i + 1]), nz = std::atoi(argv[i + 2]);
        const int cus = std::atoi(argv[3]);
        std::printf("%d\n", std::atoi(argv[2]) == 64 ? rule<double>(argv[1], nx, ny, nz, cus)
                                                     : rule<float>(argv[1], nx, ny, nz, cus));
    }
    return 0;
}
