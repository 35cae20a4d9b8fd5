// tiles.h -- geometry of the 2.5D z-marching tiles used by the fused
// Q-side kernels.  A block owns a TX x TY column of sites and marches along z
// through a chunk of planes.  Quantities needed at stencil neighbours (the
// stress, the predictor stage) are evaluated on the tile plus a one-site halo
// ring, the "evaluation plane" of PX x PY points; every thread of the block
// owns one evaluation point for the whole march (threads [0, NT) the tile's
// own sites, [NT, PN) the ring, the last few none), so its z-neighbours can
// stay in registers.  Input planes are staged in LDS with a two-site halo.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace hlb {

template <int TX_, int TY_>
struct TileShape {
    static constexpr int TX = TX_, TY = TY_;
    static constexpr int NT = TX * TY;                  // tile sites
    static constexpr int RX = TX + 4, RY = TY + 4;      // staged input plane (halo 2)
    static constexpr int RN = RX * RY;
    static constexpr int RS = (RN + 63) / 64 * 64;      // whole copies of 64 points
    static constexpr int PX = TX + 2, PY = TY + 2;      // evaluated plane (halo 1)
    static constexpr int PN = PX * PY;
    static constexpr int NH = PN - NT;                  // halo-ring points
    static constexpr int NB = (PN + 63) / 64 * 64;      // threads per block (whole waves)
    static_assert(NB <= 1024, "one evaluation point per thread");

    // Halo-ring point h in [0, NH) -> (i, j) in halo-1 plane coordinates:
    // bottom row, top row, then left/right columns.
    __host__ __device__ static __forceinline__ void halo_point(int h, int &i, int &j)
    {
        if (h < PX) {
            i = h;
            j = 0;
        } else if (h < 2 * PX) {
            i = h - PX;
            j = PY - 1;
        } else {
            const int k = h - 2 * PX;
            j = 1 + (k >> 1);
            i = (k & 1) ? PX - 1 : 0;
        }
    }
};

// The tile of the stress kernels, per precision.  FP32: 32 x 8 sites (340
// evaluation points, six waves; three blocks of the stress kernel or two of
// the fused stress and LB share a CU): the LB moves 41 values per site, and
// rows of 16 sites, 64 bytes, cost it more than the blocks gain (a 192^3 step
// 600 us where 32 x 8 takes 475).  FP64: 16 x 12 sites (252 points, four
// waves): the FP64 kernels hold about 180 and 200 registers, two waves per
// SIMD, so two four-wave blocks share a CU where a six-wave block would run
// alone with a quarter of the CU's wave slots empty.
template <typename T>
using KernelTile = typename std::conditional<sizeof(T) == 8, TileShape<16, 12>, TileShape<32, 8>>::type;

// The tile of the fused stress and LB on large lattices: 256 bytes a row, which
// the populations gain more from than the ring, 1.44 to 1.59 points a site instead
// of 1.31, costs.  FP32 steps, the narrow and the wide tile, 16 planes a chunk:
// 64^3 43 and 45 us, 128 x 64 x 64 52 and 55, 128^3 138 and 138, 192 x 192 x 64 176 and
// 150, 192^3 457 and 423, 256^3 1092 and 1035; FP64 128^3 286 and 256.
template <typename T>
using WideTile = typename std::conditional<sizeof(T) == 8, TileShape<32, 4>, TileShape<64, 5>>::type;

// z-chunk for which the tile columns S cut a lattice into fill `slots` resident
// block slots and no more (0 if the columns alone exceed them).
template <class S>
inline int fill_chunk(int nx, int ny, int nz, long long slots)
{
    const long long cols = (long long)((nx + S::TX - 1) / S::TX) * ((ny + S::TY - 1) / S::TY), chunks = slots / cols;
    return chunks < 1 ? 0 : int((nz + chunks - 1) / chunks);
}

// Whether the wide tile is taken, for chunks of tz planes.  With few sites a CU its larger
// blocks do not fill the chip: in FP64 it pays from 6000 sites a CU (128 x 128 x 100
// 257 and 226 us; 512 x 11 x 256, 5632 a CU, 195 and 203), in FP32 as well with
// chunks under 16 planes (192 x 64 x 130, 8 planes, 124 and 114; 16 planes 110 and
// 116), else from 8000 unless its blocks leave CUs idle where a CU has one of the
// others (128^3, 32 planes, 256 and 208 blocks, 145 and 156).  Its tiles may hang
// over the rows by a tenth, and its five rows cover a tenth more than the narrow
// tile's eight, a quarter more where chunks are short (512 x 6 x 512, eight rows and
// ten: 109 and 121, 123 and 123 with 8 planes).  FP32 rows that are no whole number
// of 64-byte lines cost the narrow tile more, whose every row of 32 starts or ends
// inside a line: there the wide one is taken from 6000 sites a CU and up to a third
// over (120^3 155 and 139, 150^3 377 and 310, 200^3 949 and 817, 61 x 159 x 180 172 and
// 140; whole lines: 160^3, a fifth over, 278 and 260, but 248 and 261 with 32 planes).
template <typename T>
inline bool wide_tiles(int nx, int ny, int nz, int cus, int tz)
{
    using W = WideTile<T>;
    using S = KernelTile<T>;
    const int cols = (nx + W::TX - 1) / W::TX, rows = (ny + W::TY - 1) / W::TY, chunks = (nz + tz - 1) / tz;
    const int over = cols * W::TX - nx, narrow_cols = (nx + S::TX - 1) / S::TX, narrow_rows = (ny + S::TY - 1) / S::TY;
    const bool lines = sizeof(T) == 8 || nx * sizeof(T) % 64 == 0, deep = sizeof(T) == 4 && tz >= 16;
    const long long N = (long long)nx * ny * nz;
    if ((lines ? 10 : 3) * over > nx || N < 6000LL * cus) return false;
    if (20 * rows * W::TY > (deep ? 22 : 25) * narrow_rows * S::TY) return false;
    if (!deep || !lines) return true;
    return N >= 8000LL * cus && ((long long)cols * rows * chunks >= cus || (long long)narrow_cols * narrow_rows * chunks > cus);
}

// The tile of the fused D3Q15 passes (measured at k_pc).
template <typename T>
using PassTile = typename std::conditional<sizeof(T) == 8, TileShape<32, 4>, TileShape<32, 8>>::type;

// z-chunk of the fused D3Q15 passes, or 0 where the two sweeps are the better.
// A CU evaluates its share of the blocks, each of the chunk's planes and two
// more; of the chunks that give a CU two blocks or more (all that are resident;
// with one its latencies show) the first is taken, or one with a tenth less to
// evaluate per CU.  The sites evaluated, tiles that hang over the lattice and CUs
// that wait for others included, over the sites there are tell which form is the
// faster.  A step in us with the two sweeps and with this, split coupling, FP32:
// 1.13 (128^3) 220 and 198, 1.26 (200^3) 1186 and 1157, 1.33 (96^3) 96 and 88, 1.36
// (144^3) 358 and 344 (319 and 324 with the whole-stress force), 1.40 (112^3) 144
// and 149, 1.46 (150 x 60 x 120) 117 and 124, 1.59 (140 x 100 x 100) 148 and 163;
// FP64: 1.08 (192^3) 1957 and 1592, 1.25 (144^3) 815 and 697, 1.40 (112^3) 312 and 306,
// 1.53 (300 x 50 x 120) 459 and 433.  Where a component's plane is no whole number
// of 64-byte lines the sweeps' loads and stores straddle them, and more may be
// evaluated: FP32 1.38 (61 x 159 x 127) 156 and 132, 1.43 (171 x 153 x 63) 215 and 188,
// 1.56 (54 x 165 x 113) 123 and 112, 1.70 (106 x 155 x 47) 98 and 94; FP64 1.69
// (81 x 58 x 91) 112 and 111 (107 and 104).  Tiles that hang over by more than a
// quarter are left to the sweeps (100^3, FP64, 1.44: 216 and 220), and so are chunks
// under six planes (64^3, four planes: 64 and 62, 35 and 34 in FP32).
template <typename T>
inline int pass_chunk(int nx, int ny, int nz, int cus, bool split)
{
    using S = PassTile<T>;
    const long long N = (long long)nx * ny * nz;
    const long long cols = (long long)((nx + S::TX - 1) / S::TX) * ((ny + S::TY - 1) / S::TY);
    if (cus < 1 || 4 * cols * S::NT > 5LL * nx * ny) return 0;
    int best = 0;
    long long least = 0, first = 0;  // planes a CU evaluates
    for (int c = cols < 2LL * cus ? int(2LL * cus / cols) : 1; (nz + c - 1) / c >= 6; ++c) {
        const int tz = (nz + c - 1) / c;
        const long long planes = (cols * ((nz + tz - 1) / tz) + cus - 1) / cus * (tz + 2);
        if (!best) first = planes;
        if (!best || (planes < least && 10 * planes <= 9 * first)) {
            best = tz;
            least = planes;
        }
    }
    const int most = N * sizeof(T) % 64 ? 171 : (sizeof(T) == 8 ? 155 : (split ? 138 : 135));  // percent of N
    return 100 * least * cus * S::NT <= most * N ? best : 0;
}

// The tile of the Q update, whose waves wait a third of their time (see
// k_qupdate): blocks of four waves, one to each SIMD, of which four share a CU in
// FP32 (two in FP64) and issue in turn.  In FP32 at 192^3: 32 x 8 (six waves, two blocks) 222 us,
// 32 x 12 172, 16 x 12 166 (157 with the planes copied straight into LDS);
// 24 x 7, 32 x 5, 20 x 10 and 64 x 6 were slower.
template <typename T>
using UpdateTile = TileShape<16, 12>;

__host__ __device__ __forceinline__ int wrapi(int v, int n)
{
    v %= n;
    return v < 0 ? v + n : v;
}

// Index maps of the tile kernels, shared by the kernels and the host-side
// check of their halo coverage.
template <class S>
struct TileMap {
    // Tile site t in [0, NT): its place on the halo-1 plane (pc) and on the
    // staged plane (rc).
    __host__ __device__ static __forceinline__ void own(int t, int &pc, int &rc)
    {
        const int tx = t % S::TX, ty = t / S::TX;
        pc = (ty + 1) * S::PX + (tx + 1);
        rc = (ty + 2) * S::RX + (tx + 2);
    }
    // Halo-ring point t < NH on the halo-1 plane (hp) and on the staged plane
    // (hr); -1 otherwise.
    __host__ __device__ static __forceinline__ void halo(int t, int &hp, int &hr)
    {
        hp = hr = -1;
        if (t < S::NH) {
            int i, j;
            S::halo_point(t, i, j);
            hp = j * S::PX + i;
            hr = (j + 1) * S::RX + (i + 1);
        }
    }
    // Evaluation point of thread t of a block: tile site t for t < NT, ring
    // point t - NT for NT <= t < PN (pc, rc as above); returns false, with
    // pc = rc = -1, for the threads past PN.
    __host__ __device__ static __forceinline__ bool point(int t, int &pc, int &rc)
    {
        if (t < S::NT) {
            own(t, pc, rc);
            return true;
        }
        halo(t - S::NT, pc, rc);
        return pc >= 0;
    }
    // Thread t of a block stages the elements e = t + k NB (k = 0, 1, ...) of
    // a staged plane (component-major, RN points per component).  Since
    // NB <= RN, the elements of one k lie in component comp_base(k) for
    // t < comp_split(k) and in the next one above.
    static_assert(S::NB <= S::RN, "the elements of one k span at most two components");
    __host__ __device__ static constexpr int comp_base(int k) { return k * S::NB / S::RN; }
    __host__ __device__ static constexpr int comp_split(int k) { return (comp_base(k) + 1) * S::RN - k * S::NB; }
    // Element e of an NC-component staged plane: its component and its
    // in-plane offset in the lattice for a tile at (x0, y0), periodic wrap.
    __host__ __device__ static __forceinline__ void staged(int e, int x0, int y0, int nx, int ny, int &comp, int &off)
    {
        comp = e / S::RN;
        off = staged_at(e - comp * S::RN, x0, y0, nx, ny);
    }
    // The in-plane offset of staged point r.
    __host__ __device__ static __forceinline__ int staged_at(int r, int x0, int y0, int nx, int ny)
    {
        return wrapi(x0 - 2 + r % S::RX, nx) + nx * wrapi(y0 - 2 + r / S::RX, ny);
    }
};

// Staging in chunks of 64 dwords of one component (RS values of E dwords each,
// the last RS - RN repeating the last point): which chunks the NW waves of a
// block take.  Chunk k < FULL NW of every component belongs to wave k % NW; of
// the REM chunks left over a wave takes one, for every NW/REM-th component.
template <class S, int E = 1>
struct ChunkPlan {
    static constexpr int NW = S::NB / 64, CH = S::RS * E / 64, FULL = CH / NW, REM = CH % NW;
    static constexpr int LEFT = REM > 0, STEP = REM > 0 ? NW / REM : NW;
    static_assert(REM == 0 || NW % REM == 0, "as many waves to each left-over chunk");
    // The f-th chunk of wave w (f < FULL + LEFT), and the i-th component of
    // which it takes the left-over chunk (NC and past it: none).
    __host__ __device__ static constexpr int chunk(int f, int w)
    {
        return f < FULL ? f * NW + w : FULL * NW + (REM ? w % REM : 0);
    }
    __host__ __device__ static constexpr int left_over(int i, int w, int turn)
    {
        return ((REM ? w / REM : w) + turn) % STEP + i * STEP;
    }
    // The point whose dword (chunk * 64 + lane) % E a lane copies.
    __host__ __device__ static constexpr int point(int chunk, int lane)
    {
        return (chunk * 64 + lane) / E < S::RN ? (chunk * 64 + lane) / E : S::RN - 1;
    }
};

// Block decomposition shared by the fused kernels: tiles over x and y, chunks
// of `tz` planes over z.  Consecutive logical blocks share planes, so the
// hardware block id is remapped so that each of the 8 XCDs (which receive
// workgroups round-robin) walks a contiguous range of logical blocks and
// keeps the z-halo planes in its own L2.
struct TileGrid {
    int tiles_x, tiles_y, chunks_z, tz, total, launch;
};

inline TileGrid tile_grid(int nx, int ny, int nz, int TX, int TY, int tz)
{
    TileGrid g;
    g.tiles_x = (nx + TX - 1) / TX;
    g.tiles_y = (ny + TY - 1) / TY;
    g.tz = tz;
    g.chunks_z = (nz + tz - 1) / tz;
    g.total = g.tiles_x * g.tiles_y * g.chunks_z;
    g.launch = (g.total + 7) / 8 * 8;
    return g;
}

__device__ __forceinline__ int xcd_logical_block()
{
    const int per = gridDim.x >> 3;
    return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

}  // namespace hlb
