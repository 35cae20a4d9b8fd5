// kernels.hip -- HIP kernels of the hybrid step for gfx950 and their launchers.
//
// Data layout in HBM (structure-of-arrays, component-major, x fastest):
//   g[2]  19 x N  deviation populations g_i = f_i - w_i rho0 (ping-pong, pull)
//   Q[2]   5 x N  order parameter (xx, xy, xz, yy, yz); Q[qcur] is the state,
//                 the other copy holds the predictor stage or the next Q
//   u      3 x N  velocity of the last LB step
//   Pi    12 x N  chemical stress, 9 planes (its first 3 hold F in the tiled
//                 schedule), or the 12 planes of the split coupling (sigma^xi,
//                 tau, h; see sitekern.h)
// Scalars of one run are passed by value (Coef<T>).
//
// Five schedules of one step (Sec. 2.2), chosen per lattice and precision by
// the autotuner:
//  SITES (4 sweeps, one site per thread, neighbours through L2; 95 values
//  per site cross HBM):
//   k_stress  Q^n -> Pi;  k_lb  g, div Pi -> g', u^n;
//   k_qpred   Q^n, u^n -> Q*;  k_qcorr  Q*, u^n -> Q^{n+1} (in place)
//  on small lattices in pairs (k_blb, k_bq; see small_lattice)
//  TILED (3 sweeps; the stress and the predictor stage live in LDS of 2.5D
//  z-marching tiles and are recomputed on a one-site halo ring; 65 values):
//   k_qforce  Q^n -> F^n;  k_lbf  g, F^n -> g', u^n;  k_qupdate  Q^n, u^n -> Q^{n+1}
//  MIXED (3 sweeps: the per-site stress and LB, then the tiled Q update;
//  77 values):  k_stress, k_lb, k_qupdate
//  FUSED (3 sweeps: the stress of the tiles fused with the LB step, then the
//  per-site predictor and corrector; 77 values):
//   k_qlb  Q^n, g -> g', u^n;  k_qpred;  k_qcorr
//  FUSED_TILED (2 sweeps; 59 values):  k_qlb, k_qupdate
// The split coupling (Sec. 2.2) runs the SITES and MIXED schedules with
// k_stress / k_lb writing and reading the split terms (101 and 83 values),
// and the FUSED and FUSED_TILED schedules with k_qlb<T, true>, which
// evaluates them in its tiles (77 and 59 values).
// The population sweeps (k_lb, k_lbf, k_qlb, the second D3Q15 pass k_pc2)
// load and store the populations nontemporally, and the first D3Q15 pass
// k_pc1 stores its predicted populations so (pop_load / pop_store in
// sitekern.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "order.h"
#include "site.h"
#include "sitekern.h"
#include "tiles.h"

namespace hlb {

namespace {

constexpr int BLK = 256;  // per-site kernels

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ int logical_block() { return xcd_logical_block(); }

// Fixed-order block reduction of NV doubles per thread into out[NV] (each
// round folds the upper part of the live range onto the lower one; for a
// power-of-two block this is the usual halving tree).
template <int NV, int NTH>
__device__ __forceinline__ void block_sum(double v[NV], double *out)
{
    __shared__ double buf[NV][NTH];
#pragma unroll
    for (int k = 0; k < NV; ++k) buf[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int n = NTH; n > 1;) {
        const int h = (n + 1) / 2;
        if (int(threadIdx.x) < n - h)
#pragma unroll
            for (int k = 0; k < NV; ++k) buf[k][threadIdx.x] += buf[k][threadIdx.x + h];
        __syncthreads();
        n = h;
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) out[k] = buf[k][0];
}

// Debug mode of the tiled kernels: every LDS plane is overwritten with NaN
// (by all threads, independently of the loaders' element mapping) before the
// plane is staged or evaluated into it; the caller puts a workgroup barrier
// between the fill and the writes that follow.
template <typename T>
__device__ __forceinline__ void nan_fill(T *slot, int n)
{
    const T q = __builtin_nan("");
    for (int i = int(threadIdx.x); i < n; i += int(blockDim.x)) slot[i] = q;
}

// Staging of one z-plane of an NC-component field into an LDS slot with a
// two-site halo in x and y (periodic wrap of the global coordinates) by the
// NB threads of a block.  The element -> (component, in-plane offset)
// assignment is computed once per block.
template <class Shape, int NC>
struct PlaneLoader {
    static constexpr int NE = NC * Shape::RN;
    static constexpr int NL = (NE + Shape::NB - 1) / Shape::NB;
    // only the last k has elements past the end (t >= LAST)
    static constexpr int LAST = NE - (NL - 1) * Shape::NB;
    int off[NL];  // in-plane lattice offset of the element

    __device__ __forceinline__ void init(const Geom &G, int x0, int y0)
    {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = int(threadIdx.x) + k * Shape::NB;
            int comp = 0;
            off[k] = 0;
            if (e < NE) TileMap<Shape>::staged(e, x0, y0, G.nx, G.ny, comp, off[k]);
        }
    }

    __device__ __forceinline__ static bool valid(int k) { return k < NL - 1 || int(threadIdx.x) < LAST; }

    template <typename T>
    __device__ __forceinline__ const T *elem(const T *__restrict__ src, size_t N, int plane_off, int k) const
    {
        const int cb = TileMap<Shape>::comp_base(k);
        const T *base = int(threadIdx.x) < TileMap<Shape>::comp_split(k) ? src + size_t(cb) * N : src + size_t(cb + 1) * N;
        return base + (plane_off + off[k]);
    }

    template <typename T>
    __device__ __forceinline__ void load(const T *__restrict__ src, size_t N, int plane_off,
                                         T *__restrict__ slot) const
    {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (valid(k)) slot[int(threadIdx.x) + k * Shape::NB] = *elem(src, N, plane_off, k);
    }

    // Software pipelining: issue the global loads of a plane into registers
    // now, park them in LDS after the compute of the current plane.
    template <typename T>
    __device__ __forceinline__ void fetch(const T *__restrict__ src, size_t N, int plane_off, T reg[NL]) const
    {
#pragma unroll
        for (int k = 0; k < NL; ++k) reg[k] = valid(k) ? *elem(src, N, plane_off, k) : T(0);
    }

    template <typename T>
    __device__ __forceinline__ void store(const T reg[NL], T *__restrict__ slot) const
    {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (valid(k)) slot[int(threadIdx.x) + k * Shape::NB] = reg[k];
    }
};

// Planes can go from global memory straight into LDS, 64 dwords of a component
// per instruction: no registers in between, and since the points' in-plane
// offsets are the same for every component, a wave keeps two or three of them
// and the rest of the address is scalar.  (A kernel that uses it has its LDS in
// one array: between arrays that the compiler tells apart, it waits for the
// copies before the next LDS read.)
__device__ __forceinline__ void copy4_to_lds(const char *gp, unsigned *l)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gp,
                                     (__attribute__((address_space(3))) void *)l, 4, 0, 0);
}

template <class Shape, typename T>
struct PlaneCopy {
    static constexpr int E = sizeof(T) / 4;
    using P = ChunkPlan<Shape, E>;
    unsigned off[P::FULL + P::LEFT];  // byte offset in the plane of the lane's dword of the wave's chunks
    int w;

    __device__ __forceinline__ void init(const Geom &G, int x0, int y0)
    {
        w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
        const int lane = int(threadIdx.x) & 63;
#pragma unroll
        for (int f = 0; f < P::FULL + P::LEFT; ++f) {
            const int r = P::point(P::chunk(f, w), lane);
            off[f] = unsigned(sizeof(T)) * unsigned(TileMap<Shape>::staged_at(r, x0, y0, G.nx, G.ny)) + lane % E * 4;
        }
    }
    // Issues the copy of one plane of an NC-component field into a slot of
    // stride RS; done after copies_done() of every wave and a barrier.
    template <int NC>
    __device__ __forceinline__ void issue(const T *__restrict__ src, size_t N, int plane_off, T *slot, int turn) const
    {
        auto one = [&](int c, int f) __attribute__((always_inline)) {
            copy4_to_lds(reinterpret_cast<const char *>(src + c * N + plane_off) + off[f],
                         reinterpret_cast<unsigned *>(slot + c * Shape::RS) + P::chunk(f, w) * 64);
        };
#pragma unroll
        for (int f = 0; f < P::FULL; ++f)
#pragma unroll
            for (int c = 0; c < NC; ++c) one(c, f);
        if constexpr (P::LEFT)
#pragma unroll
            for (int i = 0; i < (NC + P::STEP - 1) / P::STEP; ++i) {
                const int c = P::left_over(i, w, turn);
                if (c < NC) one(c, P::FULL);
            }
    }
};

__device__ __forceinline__ void copies_done()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), no other counter
}

// Derivatives of the 5-component Q at staged coordinate r of plane p: the
// value and its in-plane neighbours from the staged slot `mid` (two-site
// halo, RS values from one component to the next), the z-neighbours from `lo`
// (plane p-1, registers of the thread owning the point) and the staged slot
// `hi` (plane p+1).
template <class Shape, int RS, typename T>
__device__ __forceinline__ void stencil_staged(const T lo[5], const T *mid, const T *hi, int r, T q[5],
                                               T d[3][5], T lap[5])
{
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int o = k * RS + r;
        q[k] = mid[o];
        stencil7(q[k], mid[o + 1], mid[o - 1], mid[o + Shape::RX], mid[o - Shape::RX], hi[o], lo[k], d[0][k], d[1][k],
                 d[2][k], lap[k]);
    }
}

// Same for the three-slot form (all of planes p-1, p, p+1 staged).
template <class Shape, int RS, typename T>
__device__ __forceinline__ void stencil_ring(const T *lo, const T *mid, const T *hi, int r, T q[5],
                                             T d[3][5], T lap[5])
{
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int o = k * RS + r;
        q[k] = mid[o];
        stencil7(q[k], mid[o + 1], mid[o - 1], mid[o + Shape::RX], mid[o - Shape::RX], hi[o], lo[o], d[0][k], d[1][k],
                 d[2][k], lap[k]);
    }
}

// Derivatives of a 5-component field held on the evaluation plane (PX x PY,
// PN points per component) at point r: value and in-plane neighbours from
// `mid`, z-neighbours from registers.
template <class Shape, typename T>
__device__ __forceinline__ void stencil_eval(const T lo[5], const T *mid, const T hi[5], int r, T q[5],
                                             T d[3][5], T lap[5])
{
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int o = k * Shape::PN + r;
        q[k] = mid[o];
        stencil7(q[k], mid[o + 1], mid[o - 1], mid[o + Shape::PX], mid[o - Shape::PX], hi[k], lo[k], d[0][k], d[1][k],
                 d[2][k], lap[k]);
    }
}

// u and its centred gradient W_ab = d_b u_a at staged coordinate r of plane
// p: in-plane from `mid`, z from `lo` (registers, plane p-1) and `hi`.
template <class Shape, int RS, typename T>
__device__ __forceinline__ void velocity_staged(const T lo[3], const T *mid, const T *hi, int r, T uc[3],
                                                T W[3][3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int o = a * RS + r;
        uc[a] = mid[o];
        W[a][0] = T(0.5) * (mid[o + 1] - mid[o - 1]);
        W[a][1] = T(0.5) * (mid[o + Shape::RX] - mid[o - Shape::RX]);
        W[a][2] = T(0.5) * (hi[o] - lo[a]);
    }
}

struct Block {
    int x0, y0, z0, z1;
    bool ok;
};

template <class Shape>
__device__ __forceinline__ Block block_of(const Geom &G, const TileGrid &tg)
{
    Block b;
    const int lb = logical_block();
    b.ok = lb < tg.total;
    const int bx = lb % tg.tiles_x;
    const int by = (lb / tg.tiles_x) % tg.tiles_y;
    const int bz = lb / (tg.tiles_x * tg.tiles_y);
    b.x0 = bx * Shape::TX;
    b.y0 = by * Shape::TY;
    b.z0 = bz * tg.tz;
    b.z1 = min(b.z0 + tg.tz, G.nz);
    return b;
}

// ---------------------------------------------------------------- k_qforce
// F = div Pi(Q) (Eqs. (6)-(8), (19)).  Every thread owns one point of the
// evaluation plane (a tile site or a ring point).  Per plane p: evaluate the
// stress at the own point from the staged planes p-1, p, p+1 (ring points
// only where a tile site needs them), keep its z column in registers and put
// its x and y columns into one of two LDS buffers; the tile threads finish
// F(p-1) from the other buffer (the stress of plane p-1) and the z columns of
// planes p and p-2, and the plane p+2, fetched into registers at the start,
// goes into the fourth staging slot.  One barrier per plane: no slot or
// buffer is written in the plane in which it is read.  With WITH_F the block
// also sums the free-energy density of its sites.
// FP32: at most 96 registers, five waves per SIMD (three blocks per CU).  In
// FP64 (about 180 registers, two four-wave blocks per CU) a bound that would
// let a third block in spills (36 bytes per lane); with six-wave blocks such
// a bound spilled and ran slower.
template <typename T, bool WITH_F>
__global__ __launch_bounds__(KernelTile<T>::NB) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 1 : 5))) void k_qforce(Geom G, Coef<T> c, TileGrid tg,
                                                      const T *__restrict__ Q, T *__restrict__ F,
                                                      double *__restrict__ fpart, bool dbg_nan)
{
    using Shape = KernelTile<T>;
    __shared__ T sQ[4][5 * Shape::RN];
    __shared__ T sP[2][6 * Shape::PN];
    const Block B = block_of<Shape>(G, tg);
    if (!B.ok) return;
    if (dbg_nan) {
        nan_fill(&sQ[0][0], 4 * 5 * Shape::RN);
        nan_fill(&sP[0][0], 2 * 6 * Shape::PN);
        __syncthreads();
    }
    const size_t N = G.N;
    const int sxy = G.nx * G.ny;
    const int t = int(threadIdx.x);
    int pc, rc;
    const bool eval = TileMap<Shape>::point(t, pc, rc);
    const bool tile = t < Shape::NT;
    const int gx = B.x0 + t % Shape::TX, gy = B.y0 + t / Shape::TX;
    const bool mine = tile && gx < G.nx && gy < G.ny;

    PlaneLoader<Shape, 5> L;
    L.init(G, B.x0, B.y0);
    int s0 = 0, s1 = 1, s2 = 2, s3 = 3;  // s1, s2, s3: planes p-1, p, p+1; s0 free
    L.load(Q, N, wrapi(B.z0 - 2, G.nz) * sxy, sQ[s1]);
    L.load(Q, N, wrapi(B.z0 - 1, G.nz) * sxy, sQ[s2]);
    L.load(Q, N, wrapi(B.z0, G.nz) * sxy, sQ[s3]);
    __syncthreads();

    T Pz1[3] = {T(0), T(0), T(0)}, Pz2[3] = {T(0), T(0), T(0)};
    double facc = 0.0;
    constexpr int NL = PlaneLoader<Shape, 5>::NL;
    T pre[NL];
    for (int p = B.z0 - 1; p <= B.z1; ++p) {
        const bool more = p + 2 <= B.z1 + 1;
        if (more) L.fetch(Q, N, wrapi(p + 2, G.nz) * sxy, pre);
        T *Pc = sP[p & 1];        // stress of plane p (written now)
        const T *Pp = sP[~p & 1];  // stress of plane p-1 (written in the last plane)
        T Pz[3] = {T(0), T(0), T(0)};
        // ring points: only the planes whose in-plane divergence is output
        if (eval && (tile || (p >= B.z0 && p < B.z1))) {
            T q[5], d[3][5], lap[5], P[3][3], fd, H[5];
            stencil_ring<Shape, Shape::RN>(sQ[s1], sQ[s2], sQ[s3], rc, q, d, lap);
            site_stress(c, q, d, lap, P, fd, H);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Pc[a * Shape::PN + pc] = P[a][0];
                Pc[(3 + a) * Shape::PN + pc] = P[a][1];
                Pz[a] = P[a][2];
            }
            if (WITH_F && mine && p >= B.z0 && p < B.z1) facc += double(fd);
        }
        if (tile) {
            if (mine && p - 1 >= B.z0) {
                const size_t o = size_t(p - 1) * sxy + size_t(gy) * G.nx + gx;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const T Fin = (Pp[a * Shape::PN + pc + 1] - Pp[a * Shape::PN + pc - 1])
                                + (Pp[(3 + a) * Shape::PN + pc + Shape::PX] - Pp[(3 + a) * Shape::PN + pc - Shape::PX]);
                    F[a * N + o] = T(0.5) * (Fin + (Pz[a] - Pz2[a]));
                }
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Pz2[a] = Pz1[a];
                Pz1[a] = Pz[a];
            }
        }
        if (dbg_nan) {  // the free slot and the stress of plane p-1 are no longer read
            __syncthreads();
            nan_fill(sQ[s0], 5 * Shape::RN);
            nan_fill(const_cast<T *>(Pp), 6 * Shape::PN);
            __syncthreads();
        }
        if (more) L.store(pre, sQ[s0]);  // plane p+2 into the free slot
        __syncthreads();
        const int o = s0;
        s0 = s1;
        s1 = s2;
        s2 = s3;
        s3 = o;
    }
    if (WITH_F) {
        double v[1] = {facc};
        block_sum<1, Shape::NB>(v, fpart + logical_block());
    }
}

// ---------------------------------------------------------------- k_qlb
// The stress kernel fused with the LB step (Eqs. (6)-(8), (19) with the
// collision and streaming of Sec. 2.2): the plane march of k_qforce, but
// instead of writing F(p-1) each tile thread collides its site of plane p-1
// with it, pulling the populations from gin and writing gout and u^n, so F
// never goes to HBM.  The 19 pulled populations are loaded at the start of
// the plane and arrive while the stress is evaluated (loaded after it, the
// FP64 kernel ran 4% slower).
// SPLIT (Eqs. (17)-(21)): the evaluation gives sigma^xi, tau and h; the LDS
// buffers hold tau (xy, xz, yz) for the in-plane differences of the body
// force b_a = d_b tau_ab + h_a, and a tile thread keeps sigma^xi and h of its
// site of plane p-1 in registers for the collision with sigma^xi in the
// equilibrium.
// FP32: 111 registers, four waves per SIMD, two blocks per CU; FP64: about 200,
// two waves per SIMD and two four-wave blocks.  The planes of Q go straight into
// LDS (staged through registers: 127 and 231).
// Bound by memory, 46 values per site: on large lattices rows of whole lines
// matter more than the ring (see WideTile).  Q update included, FP32 192^3: 32 x 8
// tiles 457 us, 64 x 5 423 (515 with 32 x 8 tiles of both kernels staged through
// registers); 96^3 80 (86 through registers).
template <typename T, bool SPLIT, class Shape>
__global__ __launch_bounds__(Shape::NB) void k_qlb(Geom G, Coef<T> c, TileGrid tg, const T *__restrict__ Q, const T *__restrict__ gin,
                                                      T *__restrict__ gout, T *__restrict__ u, bool dbg_nan)
{
    constexpr int RS = Shape::RS;
    __shared__ T smem[4 * 5 * RS + 2 * 6 * Shape::PN];
    T(*sQ)[5 * RS] = reinterpret_cast<T(*)[5 * RS]>(smem);
    T(*sP)[6 * Shape::PN] = reinterpret_cast<T(*)[6 * Shape::PN]>(smem + 4 * 5 * RS);
    const Block B = block_of<Shape>(G, tg);
    if (!B.ok) return;
    if (dbg_nan) {
        nan_fill(&sQ[0][0], 4 * 5 * RS);
        nan_fill(&sP[0][0], 2 * 6 * Shape::PN);
        __syncthreads();
    }
    const int N = G.N;
    const int sxy = G.nx * G.ny;
    const int t = int(threadIdx.x);
    int pc, rc;
    const bool eval = TileMap<Shape>::point(t, pc, rc);
    const bool tile = t < Shape::NT;
    const int gx = B.x0 + t % Shape::TX, gy = B.y0 + t / Shape::TX;
    const bool mine = tile && gx < G.nx && gy < G.ny;

    PlaneCopy<Shape, T> L;
    L.init(G, B.x0, B.y0);
    auto stage = [&](int z, int slot) __attribute__((always_inline)) {
        L.template issue<5>(Q, size_t(N), wrapi(z, G.nz) * sxy, sQ[slot], 0);
    };
    int s0 = 0, s1 = 1, s2 = 2, s3 = 3;  // s1, s2, s3: planes p-1, p, p+1; s0 free
    stage(B.z0 - 2, s1);
    stage(B.z0 - 1, s2);
    stage(B.z0, s3);
    copies_done();
    __syncthreads();

    // z columns of the own point at planes p-1 and p-2: Pi_az, or (SPLIT) tau xz, yz
    T Pz1[3] = {T(0), T(0), T(0)}, Pz2[3] = {T(0), T(0), T(0)};
    T sig1[6], h1[3];  // SPLIT: sigma^xi and h of the own site at plane p-1
    for (int p = B.z0 - 1; p <= B.z1; ++p) {
        const bool more = p + 2 <= B.z1 + 1;
        if (more && !dbg_nan) stage(p + 2, s0);
        const bool lb = mine && p - 1 >= B.z0;  // this plane collides site (gx, gy, p-1)
        Off<T> O;
        T g[19];
        if (lb) {
            O = offsets<T>(nbr_at(G, (p - 1) * sxy + gy * G.nx + gx, gx, gy, p - 1));
#pragma unroll
            for (int i = 0; i < 19; ++i) g[i] = pop_load<true>(plane(gin, i, N), pull_off(O, CX[i], CY[i], CZ[i]));
        }
        T *Pc = sP[p & 1];         // stress (tau) of plane p (written now)
        const T *Pp = sP[~p & 1];  // stress (tau) of plane p-1 (written in the last plane)
        T Pz[3] = {T(0), T(0), T(0)};
        T sig0[6], h0[3];
        // ring points: only the planes whose in-plane divergence is used
        if (eval && (tile || (p >= B.z0 && p < B.z1))) {
            T q[5], d[3][5], lap[5], fd;
            stencil_ring<Shape, RS>(sQ[s1], sQ[s2], sQ[s3], rc, q, d, lap);
            if constexpr (SPLIT) {
                T tau3[3];
                site_split(c, q, d, lap, sig0, tau3, h0, fd);
#pragma unroll
                for (int k = 0; k < 3; ++k) Pc[k * Shape::PN + pc] = tau3[k];
                Pz[0] = tau3[1];
                Pz[1] = tau3[2];
            } else {
                T P[3][3], H[5];
                site_stress(c, q, d, lap, P, fd, H);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    Pc[a * Shape::PN + pc] = P[a][0];
                    Pc[(3 + a) * Shape::PN + pc] = P[a][1];
                    Pz[a] = P[a][2];
                }
            }
        }
        copies_done();  // and the populations, ahead of the stores, which are not waited for
        if (tile) {
            if (lb) {
                T f[3], uu[3], rho;
                if constexpr (SPLIT) {
                    // b_a = d_b tau_ab + h_a at plane p-1: in-plane differences from LDS,
                    // z differences from the own point's tau at planes p and p-2
                    const T *txy = Pp, *txz = Pp + Shape::PN, *tyz = Pp + 2 * Shape::PN;
                    f[0] = T(0.5) * ((txy[pc + Shape::PX] - txy[pc - Shape::PX]) + (Pz[0] - Pz2[0])) + h1[0];
                    f[1] = T(0.5) * ((Pz[1] - Pz2[1]) - (txy[pc + 1] - txy[pc - 1])) + h1[1];
                    f[2] = T(0.5) * (-(txz[pc + 1] - txz[pc - 1]) - (tyz[pc + Shape::PX] - tyz[pc - Shape::PX])) +
                           h1[2];
                    lb_collide_split(c, g, f, sig1, uu, rho);
                } else {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        const T Fin = (Pp[a * Shape::PN + pc + 1] - Pp[a * Shape::PN + pc - 1])
                                    + (Pp[(3 + a) * Shape::PN + pc + Shape::PX] - Pp[(3 + a) * Shape::PN + pc - Shape::PX]);
                        f[a] = T(0.5) * (Fin + (Pz[a] - Pz2[a]));
                    }
                    lb_collide(c, g, f, uu, rho);
                }
#pragma unroll
                for (int i = 0; i < 19; ++i) pop_store<true>(plane(gout, i, N), O.s, g[i]);
#pragma unroll
                for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Pz2[a] = Pz1[a];
                Pz1[a] = Pz[a];
            }
            if constexpr (SPLIT) {
#pragma unroll
                for (int k = 0; k < 6; ++k) sig1[k] = sig0[k];
#pragma unroll
                for (int a = 0; a < 3; ++a) h1[a] = h0[a];
            }
        }
        if (dbg_nan) {  // the free slot and the stress of plane p-1 are no longer read
            __syncthreads();
            nan_fill(sQ[s0], 5 * RS);
            nan_fill(const_cast<T *>(Pp), 6 * Shape::PN);
            __syncthreads();
            if (more) stage(p + 2, s0);
            copies_done();
        }
        __syncthreads();
        const int o = s0;
        s0 = s1;
        s1 = s2;
        s2 = s3;
        s3 = o;
    }
}

// ---------------------------------------------------------------- k_qupdate
// Predictor-corrector for the Q equation with u held at u^n (Eqs. (2)-(4)):
//   Q* = Q + R(Q, u),  Q' = [Q + Q* + R(Q*, u)] / 2   (= Q + [R(Q) + R(Q*)]/2).
// Every thread owns one point of the evaluation plane.  Per plane p: the
// predictor stage Q*(p) at the own point (in-plane stencil from the staged
// plane p, z-neighbours from the registers holding Q(p-1), u(p-1) and the
// staged plane p+1; ring points only where a tile site needs them); then on
// the tile threads the corrector at plane p-1 from Q*(p-1) in LDS and
// Q*(p-2), Q*(p) in registers, with u(p-1) and W(p-1) kept from the
// predictor of plane p-1.  Q*(p) goes into the other of two LDS buffers and the
// plane p+2 is copied into the third staging slot meanwhile, so a plane takes
// one barrier.  FP32: 127 registers and 40.8 kB, four blocks a CU; FP64: 208
// and 81.6 kB, two.
// Bound neither by issue nor by memory alone: of its time at 128^3 vector issue
// takes 0.58 in FP32 and 0.36 in FP64 (about 450 instructions a point and plane, of
// which the ring and the two extra planes of a chunk repeat half), its 142 and 270 MB
// at the rate of a copy 0.44 and 0.47, and a resident wave spends 0.37 and 0.34 in
// waits (LDS, the copies, the barrier of a plane) and 0.17 and 0.20 for an issue slot.
// FP32 at 192^3: 222 us with 32 x 8 tiles staged through registers, 160 us now (590
// MB of Q and u, 3.7 TB/s); at 128^3 65 and 53 us, where k_qpred and k_qcorr take 47.
// FP64, staged through registers into two slots and one buffer with two barriers a
// plane: 96^3 55 us and now 46, 128^3 97 and 97, 192^3 297 and 279.
template <typename T>
__global__ __launch_bounds__(UpdateTile<T>::NB) void k_qupdate(Geom G, Coef<T> c, TileGrid tg,
                                                       const T *__restrict__ Qin, const T *__restrict__ u,
                                                       T *__restrict__ Qout, bool dbg_nan)
{
    using Shape = UpdateTile<T>;
    constexpr int NQS = 3, NSS = 2, RS = Shape::RS;
    __shared__ T smem[NQS * 8 * RS + NSS * 5 * Shape::PN];
    T(*sQ)[5 * RS] = reinterpret_cast<T(*)[5 * RS]>(smem);
    T(*sU)[3 * RS] = reinterpret_cast<T(*)[3 * RS]>(smem + NQS * 5 * RS);
    T(*sS)[5 * Shape::PN] = reinterpret_cast<T(*)[5 * Shape::PN]>(smem + NQS * 8 * RS);
    const Block B = block_of<Shape>(G, tg);
    if (!B.ok) return;
    if (dbg_nan) {
        nan_fill(&sQ[0][0], NQS * 5 * RS);
        nan_fill(&sU[0][0], NQS * 3 * RS);
        nan_fill(&sS[0][0], NSS * 5 * Shape::PN);
        __syncthreads();
    }
    const size_t N = G.N;
    const int sxy = G.nx * G.ny;
    const int t = int(threadIdx.x);
    int pc, rc;
    const bool eval = TileMap<Shape>::point(t, pc, rc);
    const bool tile = t < Shape::NT;
    const int gx = B.x0 + t % Shape::TX, gy = B.y0 + t / Shape::TX;
    const bool mine = tile && gx < G.nx && gy < G.ny;

    int sc = 0, sn = 1, sf = 2;  // slots of planes p, p+1 and the free one
    PlaneCopy<Shape, T> L;
    L.init(G, B.x0, B.y0);
    auto stage = [&](int z, int slot) __attribute__((always_inline)) {
        const int o = wrapi(z, G.nz) * sxy;
        L.template issue<5>(Qin, N, o, sQ[slot], 0);
        L.template issue<3>(u, N, o, sU[slot], PlaneCopy<Shape, T>::P::STEP - 1);
    };
    stage(B.z0 - 1, sc);
    stage(B.z0, sn);
    // Plane state of the own point in two register sets: one holds Q, u and,
    // on tile sites, W of plane p-1, the other receives those of plane p.  In
    // FP32 they swap roles from one plane to the next (the loop below is
    // unrolled by two); in FP64 the new set is copied over the old.  First Q
    // and u of plane z0 - 2 (the ring's first predictor is at plane z0).
    T qA[5] = {T(0), T(0), T(0), T(0), T(0)}, uA[3] = {T(0), T(0), T(0)}, WA[3][3], qB[5], uB[3], WB[3][3];
    if (tile) {
        const int o = wrapi(B.z0 - 2, G.nz) * sxy + wrapi(B.x0 - 2 + rc % Shape::RX, G.nx)
                    + G.nx * wrapi(B.y0 - 2 + rc / Shape::RX, G.ny);
#pragma unroll
        for (int k = 0; k < 5; ++k) qA[k] = Qin[size_t(k) * N + o];
#pragma unroll
        for (int a = 0; a < 3; ++a) uA[a] = u[size_t(a) * N + o];
    }
    copies_done();
    __syncthreads();

    T qs2[5] = {T(0), T(0), T(0), T(0), T(0)};  // Q* at the own site, plane p-2
    auto plane = [&](int p, const T (&qmm)[5], const T (&umm)[3], const T (&Wmm)[3][3], T (&q0)[5], T (&u0)[3],
                     T (&W0)[3][3]) __attribute__((always_inline)) {
        const bool more = p + 2 <= B.z1 + 1;
        if (more && !dbg_nan) stage(p + 2, sf);
        T qs0[5];
        T *Scur = sS[p & 1];         // receives Q*(p)
        const T *Sprev = sS[~p & 1];  // holds Q*(p-1)
        if (eval) {
#pragma unroll
            for (int k = 0; k < 5; ++k) q0[k] = sQ[sc][k * RS + rc];
#pragma unroll
            for (int a = 0; a < 3; ++a) u0[a] = sU[sc][a * RS + rc];
        }
        const bool pred = eval && (tile || (p >= B.z0 && p < B.z1));
        if (pred) {
            T q[5], d[3][5], lap[5], uc[3], R[5];
            stencil_staged<Shape, RS>(qmm, sQ[sc], sQ[sn], rc, q, d, lap);
            velocity_staged<Shape, RS>(umm, sU[sc], sU[sn], rc, uc, W0);
            site_rhs(c, q, d, lap, uc, W0, R);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                qs0[k] = q[k] + R[k];
                Scur[k * Shape::PN + pc] = qs0[k];
            }
        }
        T out[5];
        if (tile && p - 1 >= B.z0) {
            T q[5], d[3][5], lap[5], R[5];
            stencil_eval<Shape>(qs2, Sprev, qs0, pc, q, d, lap);
            site_rhs(c, q, d, lap, umm, Wmm, R);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                out[k] = T(0.5) * (qmm[k] + q[k] + R[k]);
                qs2[k] = q[k];
                asm volatile("" : "+v"(out[k]));  // evaluated here, not after the wait below
            }
        } else if (tile && p == B.z0) {
            // Q*(z0 - 1) is not corrected but is the z-neighbour of the corrector at z0
#pragma unroll
            for (int k = 0; k < 5; ++k) qs2[k] = Sprev[k * Shape::PN + pc];
        }
        copies_done();  // ahead of the stores, which are not waited for
        if (mine && p - 1 >= B.z0) {
            const size_t o = size_t(p - 1) * sxy + size_t(gy) * G.nx + gx;
#pragma unroll
            for (int k = 0; k < 5; ++k) Qout[k * N + o] = out[k];
        }
        if (dbg_nan) {  // the free slots and Q*(p-1) are no longer read
            __syncthreads();
            nan_fill(sQ[sf], 5 * RS);
            nan_fill(sU[sf], 3 * RS);
            nan_fill(const_cast<T *>(Sprev), 5 * Shape::PN);
            __syncthreads();
            if (more) stage(p + 2, sf);
            copies_done();
        }
        __syncthreads();
        const int o = sc;
        sc = sn;
        sn = sf;
        sf = o;
    };
    int p = B.z0 - 1;
    if constexpr (sizeof(T) == 4) {
        for (; p <= B.z1; p += 2) {
            plane(p, qA, uA, WA, qB, uB, WB);
            // an odd plane by this copy of the code too: one of its own would fuse other products
            if (p + 1 > B.z1) break;
            plane(p + 1, qB, uB, WB, qA, uA, WA);
        }
    } else {
        // FP64: a second copy of the plane code costs more registers than the
        // copies of the plane state it saves
        for (; p <= B.z1; ++p) {
            plane(p, qA, uA, WA, qB, uB, WB);
#pragma unroll
            for (int k = 0; k < 5; ++k) qA[k] = qB[k];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                uA[a] = uB[a];
#pragma unroll
                for (int b2 = 0; b2 < 3; ++b2) WA[a][b2] = WB[a][b2];
            }
        }
    }
}

// ---------------------------------------------------------------- per-site kernels

template <int B = BLK>
__device__ __forceinline__ int site_index() { return logical_block() * B + int(threadIdx.x); }

// SPLIT: the 12 planes of the split coupling instead of the 9 of Pi.
// Occupancy floors of the per-site Q-side kernels in FP64 (blocks of 256 per
// CU): registers bounded to 128 (stress, corrector) and 96 (predictor)
// without spills, 4 and 5 waves per SIMD.  FP32 is left to the compiler
// (~60 registers, 8 waves).
template <typename T, bool SPLIT, int B = BLK>
__global__ __launch_bounds__(B, sizeof(T) == 8 ? 4 : 1) void k_stress(Geom G, Coef<T> c, const T *__restrict__ Q,
                                                T *__restrict__ Pi, double *__restrict__ fpart)
{
    const int s = site_index<B>();
    double fsum = 0.0;
    if (s < G.N) fsum = double(SPLIT ? split_at(G, c, Q, Pi, s) : stress_at(G, c, Q, Pi, s));
    if (fpart) {
        double v[1] = {fsum};
        block_sum<1, B>(v, fpart + logical_block());
    }
}

template <typename T, bool SPLIT, int B>
__global__ __launch_bounds__(B) void k_lb(Geom G, Coef<T> c, const T *__restrict__ gin,
                                            const T *__restrict__ Pi, T *__restrict__ gout, T *__restrict__ u)
{
    const int s = site_index<B>();
    if (s >= G.N) return;
    if (SPLIT)
        lb_split_at<T, true>(G, c, gin, Pi, gout, u, s);
    else
        lb_at<T, true>(G, c, gin, Pi, gout, u, s);
}

template <typename T, int B>
__global__ __launch_bounds__(B, sizeof(T) == 8 ? 5 : 1) void k_qpred(Geom G, Coef<T> c, const T *__restrict__ Q,
                                               const T *__restrict__ u, T *__restrict__ Qs)
{
    const int s = site_index<B>();
    if (s < G.N) pred_at(G, c, Q, u, Qs, s);
}

template <typename T, int B>
__global__ __launch_bounds__(B, sizeof(T) == 8 ? 4 : 1) void k_qcorr(Geom G, Coef<T> c, T *__restrict__ Q, const T *__restrict__ Qs,
                                               const T *__restrict__ u)
{
    const int s = site_index<B>();
    if (s < G.N) corr_at(G, c, Q, Qs, u, s);
}

// The same, two sites per thread (nx even), in FP64: a wave's load of one value
// per lane is 512 bytes there, and the 61 to 66 of them that a site takes in k_qpred
// and k_qcorr fill a CU's path to its cache; two sites a thread take 56 to 61 of
// twice the width and no shifted rows.  About 235 registers, two waves per SIMD.
// Both together at 96^3 57 -> 45 us, 128^3 123 -> 100 (520 MB if nothing is cached:
// the memory's rate), 64^3 21 -> 17.  In FP32 they are slower (128^3 52 -> 58): one
// value per lane is at the memory's rate already, with four times the waves.
template <typename T, int B>
__global__ __launch_bounds__(B) void k_qpred2(Geom G, Coef<T> c, const T *__restrict__ Q, const T *__restrict__ u,
                                              T *__restrict__ Qs)
{
    const int p = site_index<B>();
    pred_pair(G, c, Q, u, Qs, 2 * min(p, G.N / 2 - 1), p < G.N / 2);
}

template <typename T, int B>
__global__ __launch_bounds__(B) void k_qcorr2(Geom G, Coef<T> c, T *__restrict__ Q, const T *__restrict__ Qs,
                                              const T *__restrict__ u)
{
    const int p = site_index<B>();
    corr_pair(G, c, Q, Qs, u, 2 * min(p, G.N / 2 - 1), p < G.N / 2);
}

// ---------------------------------------------------------------- small lattices
// The per-site sweeps in pairs, over bricks of sites: k_blb is k_stress and
// k_lb, k_bq is k_qpred and k_qcorr.  A block evaluates the first of the two on
// its brick and the brick's six faces, one point per thread, into LDS, and the
// second on the brick out of LDS; the stencils come from global memory as in
// the per-site sweeps, whose arithmetic these repeat.  That is about
// twice the evaluations, but on a lattice that does not fill the chip a kernel
// takes 3.5 us or more, whatever it computes, and a step has two of them instead
// of four (see small_lattice).
template <int BX_, int BY_, int BZ_>
struct Brick {
    static constexpr int BX = BX_, BY = BY_, BZ = BZ_;
    static constexpr int NT = BX * BY * BZ;                                     // sites, the first threads
    static constexpr int FX = 2 * BY * BZ, FY = 2 * BX * BZ, FZ = 2 * BX * BY;  // face points
    static constexpr int NP = NT + FX + FY + FZ, NB = (NP + 63) / 64 * 64;      // points; threads
    static constexpr int PX = BX + 2, PY = BY + 2, PN = PX * PY * (BZ + 2);     // plane of a value in LDS
    static_assert(NB <= 1024, "one point per thread");

    // Thread t's point (t < NP): coordinates in the brick, -1 and BX, BY, BZ on the faces.
    __device__ static __forceinline__ void point(int t, int &i, int &j, int &k)
    {
        if (t < NT) {
            i = t % BX;
            j = t / BX % BY;
            k = t / (BX * BY);
        } else if ((t -= NT) < FX) {
            j = t % BY;
            k = t / BY % BZ;
            i = t < FX / 2 ? -1 : BX;
        } else if ((t -= FX) < FY) {
            i = t % BX;
            k = t / BX % BZ;
            j = t < FY / 2 ? -1 : BY;
        } else {
            t -= FY;
            i = t % BX;
            j = t / BX % BY;
            k = t < FZ / 2 ? -1 : BZ;
        }
    }
    static int blocks(const Geom &G)
    {
        return ((G.nx + BX - 1) / BX) * ((G.ny + BY - 1) / BY) * ((G.nz + BZ - 1) / BZ);
    }
};

// The point of a thread: its site and neighbours (periodic; where the brick
// hangs over the lattice past its first halo plane any site does), its place in
// an LDS plane, and whether it is a site of the brick.
struct BrickPoint {
    Nbr S;
    int p;
    bool mine;
};

template <class B>
__device__ __forceinline__ BrickPoint brick_point(const Geom &G, int block)
{
    const int nbx = (G.nx + B::BX - 1) / B::BX, nby = (G.ny + B::BY - 1) / B::BY;
    const int r = block / nbx, bz = r / nby;
    int i, j, k;
    // the threads past the last point repeat it (same values to the same places)
    B::point(min(int(threadIdx.x), B::NP - 1), i, j, k);
    int x = (block - r * nbx) * B::BX + i, y = (r - bz * nby) * B::BY + j, z = bz * B::BZ + k;
    BrickPoint b;
    b.mine = int(threadIdx.x) < B::NT && x < G.nx && y < G.ny && z < G.nz;
    b.p = ((k + 1) * B::PY + j + 1) * B::PX + i + 1;
    auto wrap1 = [](int v, int n) __attribute__((always_inline)) {
        v += v < 0 ? n : 0;
        v -= v >= n ? n : 0;
        return min(v, n - 1);
    };
    x = wrap1(x, G.nx);
    y = wrap1(y, G.ny);
    z = wrap1(z, G.nz);
    b.S = nbr_at(G, x + G.nx * (y + G.ny * z), x, y, z);
    return b;
}

template <typename T, bool SPLIT, class B>
__global__ __launch_bounds__(B::NB) void k_blb(Geom G, Coef<T> c, int nblocks, const T *__restrict__ Q,
                                               const T *__restrict__ gin, T *__restrict__ gout, T *__restrict__ u)
{
    constexpr int PN = B::PN, DX = 1, DY = B::PX, DZ = B::PX * B::PY;
    __shared__ T sP[SPLIT ? 3 : 9][PN];
    const int block = logical_block();
    if (block >= nblocks) return;
    const BrickPoint b = brick_point<B>(G, block);
    const int N = G.N, p = b.p;
    const Off<T> O = offsets<T>(b.S);
    T g[19];
    if (b.mine)
#pragma unroll
        for (int i = 0; i < 19; ++i) g[i] = pop_load<false>(plane(gin, i, N), pull_off(O, CX[i], CY[i], CZ[i]));
    T q[5], d[3][5], lap[5], fd, sig[6], h[3];
    gather_q(Q, N, O, q, d, lap);
    if constexpr (SPLIT) {
        T tau3[3];
        site_split(c, q, d, lap, sig, tau3, h, fd);
#pragma unroll
        for (int k = 0; k < 3; ++k) sP[k][p] = tau3[k];
    } else {
        T P[3][3], H[5];
        site_stress(c, q, d, lap, P, fd, H);
#pragma unroll
        for (int k = 0; k < 9; ++k) sP[k][p] = P[k / 3][k % 3];
    }
    __syncthreads();
    if (!b.mine) return;
    T f[3], uu[3], rho;
    if constexpr (SPLIT) {
        const T *txy = sP[0], *txz = sP[1], *tyz = sP[2];
        f[0] = T(0.5) * ((txy[p + DY] - txy[p - DY]) + (txz[p + DZ] - txz[p - DZ])) + h[0];
        f[1] = T(0.5) * ((tyz[p + DZ] - tyz[p - DZ]) - (txy[p + DX] - txy[p - DX])) + h[1];
        f[2] = T(0.5) * (-(txz[p + DX] - txz[p - DX]) - (tyz[p + DY] - tyz[p - DY])) + h[2];
        lb_collide_split(c, g, f, sig, uu, rho);
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            f[a] = T(0.5) * ((sP[3 * a][p + DX] - sP[3 * a][p - DX]) + (sP[3 * a + 1][p + DY] - sP[3 * a + 1][p - DY]) +
                             (sP[3 * a + 2][p + DZ] - sP[3 * a + 2][p - DZ]));
        lb_collide(c, g, f, uu, rho);
    }
#pragma unroll
    for (int i = 0; i < 19; ++i) pop_store<false>(plane(gout, i, N), O.s, g[i]);
#pragma unroll
    for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
}

template <typename T, class B>
__global__ __launch_bounds__(B::NB) void k_bq(Geom G, Coef<T> c, int nblocks, const T *__restrict__ Q,
                                              const T *__restrict__ u, T *__restrict__ Qout)
{
    constexpr int PN = B::PN, DX = 1, DY = B::PX, DZ = B::PX * B::PY;
    __shared__ T sS[5][PN];
    const int block = logical_block();
    if (block >= nblocks) return;
    const BrickPoint b = brick_point<B>(G, block);
    const int N = G.N, p = b.p;
    const Off<T> O = offsets<T>(b.S);
    T qn[5], q[5], d[3][5], lap[5], uc[3], V[3][3], W[3][3], R[5];
    gather_q(Q, N, O, qn, d, lap);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T *P = plane(u, a, N);
        uc[a] = *at(P, O.s);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            V[a][e] = *at(P, O.nb[2 * e]) - *at(P, O.nb[2 * e + 1]);
            W[a][e] = T(0.5) * V[a][e];
        }
    }
    site_rhs(c, qn, d, lap, uc, W, R);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        q[k] = qn[k] + R[k];
        sS[k][p] = q[k];
    }
    __syncthreads();
    if (!b.mine) return;
    // The gradient once more from the differences, which the compiler may not
    // trace back: shared between the two stages, its products would be fused
    // otherwise than in k_qpred and k_qcorr.
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            asm volatile("" : "+v"(V[a][e]));
            W[a][e] = T(0.5) * V[a][e];
        }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const T *P = sS[k] + p;
        stencil7(q[k], P[DX], P[-DX], P[DY], P[-DY], P[DZ], P[-DZ], d[0][k], d[1][k], d[2][k], lap[k]);
    }
    site_rhs(c, q, d, lap, uc, W, R);
#pragma unroll
    for (int k = 0; k < 5; ++k) *at(plane(Qout, k, N), O.s) = T(0.5) * (qn[k] + q[k] + R[k]);
}

// D3Q15 predictor-corrector LB, the two passes (see pc1_at, pc2_at).
template <typename T, bool SPLIT, int B>
__global__ __launch_bounds__(B) void k_pc1(Geom G, Coef<T> c, const T *__restrict__ g, const T *__restrict__ Pi,
                                             T *__restrict__ P, T *__restrict__ u, T *__restrict__ bsave)
{
    const int s = site_index<B>();
    if (s < G.N) pc1_at<T, SPLIT, true>(G, c, g, Pi, P, u, bsave, s);
}

template <typename T, bool SPLIT, int B>
__global__ __launch_bounds__(B) void k_pc2(Geom G, Coef<T> c, const T *__restrict__ g, const T *__restrict__ P,
                                             const T *__restrict__ Pi, const T *__restrict__ bsave,
                                             T *__restrict__ gout)
{
    const int s = site_index<B>();
    if (s < G.N) pc2_at<T, SPLIT, true>(G, c, g, P, Pi, bsave, gout, s);
}

// Both passes in one sweep: the block marches along z as the tile kernels do,
// with one point of the evaluation plane (tile and ring, corners included) per
// thread.  Per plane p: the first pass at the own point, f and P = f + C into
// LDS for the twelve velocities that move in the plane (rest and z stay in the
// column's registers); then the tile threads pull: velocities with e_z = -1
// arriving in plane p-1, which completes f* there and lets the second pass
// write the site, those with e_z = 0 for plane p, and e_z = 1 for plane p+1.
// Pulled pairs are carried as f* and (f + P)/2.  P and the saved force never
// go to HBM: 45 values per site instead of 102.  One LDS buffer and two barriers
// a plane; 99 registers in FP32, about 200 in FP64, two blocks a CU.
// Bound by the path from the cache (36 loads a point and plane) and by latency:
// 114 us at 128^3 in FP32, where k_pc1 and k_pc2 take 132.  A step in us with the
// two passes and with this, split coupling: 128^3 219 and 197 (with 64 x 5 tiles 5
// more, 32 x 4 21, 16 x 12 46), in FP64 521 and 433 (16 x 12 13 more); 96^3 97 and 88,
// 203 and 175.
template <typename T, bool SPLIT>
__global__ __launch_bounds__(PassTile<T>::NB) void k_pc(Geom G, Coef<T> c, TileGrid tg, const T *__restrict__ g,
                                                         const T *__restrict__ Pi, T *__restrict__ gout,
                                                         T *__restrict__ u)
{
    using Shape = PassTile<T>;
    constexpr int PN = Shape::PN, PX = Shape::PX;
    __shared__ T S[2][12][PN];  // f and P
    const Block B = block_of<Shape>(G, tg);
    if (!B.ok) return;
    const int N = G.N, sxy = G.nx * G.ny;
    // the threads past the last point repeat it (same values to the same places)
    int pc, rc;
    TileMap<Shape>::point(min(int(threadIdx.x), PN - 1), pc, rc);
    const int x = wrapi(B.x0 + pc % PX - 1, G.nx), y = wrapi(B.y0 + pc / PX - 1, G.ny);
    const bool mine = int(threadIdx.x) < Shape::NT && B.x0 + pc % PX - 1 < G.nx && B.y0 + pc / PX - 1 < G.ny;
    // f* and (f + P)/2 arriving at the own site: in plane p-1 (e_z = 1 and 0) and plane p (e_z = 1)
    T as[15], ao[15], ns[15], no[15], b1[3], sig1[6];
    for (int p = B.z0 - 1; p <= B.z1; ++p) {
        const int z = wrapi(p, G.nz);
        const Off<T> O = offsets<T>(nbr_at(G, x + G.nx * y + z * sxy, x, y, z));
        T f[15], C[15], b[3], sig[6], uu[3], rho;
#pragma unroll
        for (int i = 0; i < 15; ++i) f[i] = *at(plane(g, i, N), O.s);
        force15<T, SPLIT>(Pi, N, O, b, sig);
        lb15_collide<T, SPLIT>(c, f, sig, b, C, uu, rho);
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            C[i] += f[i];
            if (DX15[i] || DY15[i]) {
                const int k = i < 5 ? i - 1 : i - 3;
                S[0][k][pc] = f[i];
                S[1][k][pc] = C[i];
            }
        }
        if (mine && p >= B.z0 && p < B.z1)
#pragma unroll
            for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
        __syncthreads();
        if (mine) {
            auto pull = [&](int i, T &fs, T &fo) __attribute__((always_inline)) {
                T f0 = f[i];
                fs = C[i];
                if (DX15[i] || DY15[i]) {
                    const int k = i < 5 ? i - 1 : i - 3, o = pc - DX15[i] - PX * DY15[i];
                    f0 = S[0][k][o];
                    fs = S[1][k][o];
                }
                fo = T(0.5) * (f0 + fs);
            };
            if (p > B.z0) {
#pragma unroll
                for (int i = 0; i < 15; ++i)
                    if (DZ15[i] < 0) pull(i, as[i], ao[i]);
                T D[15], u2[3], rho2;
                lb15_collide<T, SPLIT>(c, as, sig1, b1, D, u2, rho2);
                const unsigned o = unsigned(x + G.nx * y + (p - 1) * sxy) * unsigned(sizeof(T));
#pragma unroll
                for (int i = 0; i < 15; ++i) pop_store<true>(plane(gout, i, N), o, fmat(T(0.5), D[i], ao[i]));
            }
#pragma unroll
            for (int i = 0; i < 15; ++i) {
                if (DZ15[i] == 0) pull(i, as[i], ao[i]);
                if (DZ15[i] > 0) {
                    as[i] = ns[i];
                    ao[i] = no[i];
                    pull(i, ns[i], no[i]);
                }
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) b1[a] = b[a];
            if constexpr (SPLIT)
#pragma unroll
                for (int k = 0; k < 6; ++k) sig1[k] = sig[k];
        }
        __syncthreads();
    }
}

// D3Q15 state from (rho, u): g_i(x) = f_i^eq(rho(x), u(x)) - A_s(rho0) in
// place, without stress or force terms; Q converted to the storage type.
template <typename T>
__global__ __launch_bounds__(BLK) void k_init15(Geom G, Coef<T> c, const double *__restrict__ rho_in,
                                                const double *__restrict__ u_in, const double *__restrict__ Q_in,
                                                T *__restrict__ g, T *__restrict__ Q)
{
    const int s = site_index();
    if (s >= G.N) return;
    const size_t N = G.N;
    const T uu3[3] = {T(u_in[s]), T(u_in[N + s]), T(u_in[2 * N + s])};
    const T uu = uu3[0] * uu3[0] + uu3[1] * uu3[1] + uu3[2] * uu3[2];
#pragma unroll
    for (int i = 0; i < 15; ++i) g[i * N + s] = lb15_eq(i, c.rho0, T(rho_in[s]), uu3, uu);
#pragma unroll
    for (int k = 0; k < 5; ++k) Q[k * N + s] = T(Q_in[k * N + s]);
}

// D3Q15 readout: rho and u = sum f e / rho of the stored populations
// (Eq. (14); u == 0 with the flow off), Q in FP64, FP64 block partials.
template <typename T>
__global__ __launch_bounds__(BLK) void k_readout15(Geom G, Coef<T> c, const T *__restrict__ g, bool flow,
                                                   const T *__restrict__ Q, double *__restrict__ rho_out,
                                                   double *__restrict__ u_out, double *__restrict__ Q_out,
                                                   double *__restrict__ part)
{
    const int s = site_index();
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (s < G.N) {
        const size_t N = G.N;
        T drho = T(0), j[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            const T f = g[i * N + s];
            drho += f;
            j[0] += T(DX15[i]) * f;
            j[1] += T(DY15[i]) * f;
            j[2] += T(DZ15[i]) * f;
        }
        const T rho = c.rho0 + drho;
        if (rho_out) rho_out[s] = double(rho);
        if (u_out)
#pragma unroll
            for (int a = 0; a < 3; ++a) u_out[a * N + s] = flow ? double(j[a] / rho) : 0.0;
        if (Q_out)
#pragma unroll
            for (int k = 0; k < 5; ++k) Q_out[k * N + s] = double(Q[k * N + s]);
        v[0] = double(drho);
        if (flow)
#pragma unroll
            for (int a = 0; a < 3; ++a) v[1 + a] = double(j[a]);
    }
    if (part) block_sum<4, BLK>(v, part + 4 * logical_block());
}

// LB with a precomputed body force (tiled schedule).
template <typename T>
__global__ __launch_bounds__(BLK) void k_lbf(Geom G, Coef<T> c, const T *__restrict__ gin,
                                             const T *__restrict__ F, T *__restrict__ gout, T *__restrict__ u)
{
    const int s = site_index();
    if (s >= G.N) return;
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T g[19], f[3], uu[3], rho;
#pragma unroll
    for (int i = 0; i < 19; ++i) g[i] = pop_load<true>(plane(gin, i, N), pull_off(O, CX[i], CY[i], CZ[i]));
#pragma unroll
    for (int a = 0; a < 3; ++a) f[a] = *at(plane(F, a, N), O.s);
    lb_collide(c, g, f, uu, rho);
#pragma unroll
    for (int i = 0; i < 19; ++i) pop_store<true>(plane(gout, i, N), O.s, g[i]);
#pragma unroll
    for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
}

// Populations such that the first pull returns g^eq(rho(x), u(x)):
// g_i(y) = g_i^eq(rho(y + e_i), u(y + e_i)); Q converted to the storage type.
template <typename T>
__global__ __launch_bounds__(BLK) void k_init(Geom G, Coef<T> c, const double *__restrict__ rho_in,
                                              const double *__restrict__ u_in,
                                              const double *__restrict__ Q_in, T *__restrict__ g,
                                              T *__restrict__ Q)
{
    const int s = site_index();
    if (s >= G.N) return;
    const size_t N = G.N;
    const Nbr S = nbr_of(G, s);
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const int t = pull_from(G, S, -CX[i], -CY[i], -CZ[i]);
        const T uu[3] = {T(u_in[t]), T(u_in[N + t]), T(u_in[2 * N + t])};
        g[i * N + s] = lb_geq(c, i, T(rho_in[t]), uu);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) Q[k * N + s] = T(Q_in[k * N + s]);
}

// Current-level readout: rho, u = (j + F/2)/rho with F = div Pi, or the split
// body force b (u == 0 when Pi is null, i.e. flow off) and Q in FP64; FP64
// block partials of (rho - rho0, rho u_x, rho u_y, rho u_z).
template <typename T, bool SPLIT>
__global__ __launch_bounds__(BLK) void k_readout(Geom G, Coef<T> c, const T *__restrict__ g,
                                                 const T *__restrict__ Pi, const T *__restrict__ Q,
                                                 double *__restrict__ rho_out, double *__restrict__ u_out,
                                                 double *__restrict__ Q_out, double *__restrict__ part)
{
    const int s = site_index();
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (s < G.N) {
        const size_t N = G.N;
        const Nbr S = nbr_of(G, s);
        T gg[19], drho, j[3], f[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int i = 0; i < 19; ++i) gg[i] = g[i * N + pull_from(G, S, CX[i], CY[i], CZ[i])];
        lb_moments(gg, drho, j);
        if (Pi) {
            const Off<T> O = offsets<T>(S);
            if (SPLIT)
                split_force(Pi, G.N, O, f);
            else
                divergence(Pi, G.N, O, f);
        }
        const T rho = c.rho0 + drho;
        T uu[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) uu[a] = Pi ? (j[a] + T(0.5) * f[a]) / rho : T(0);
        if (rho_out) rho_out[s] = double(rho);
        if (u_out)
#pragma unroll
            for (int a = 0; a < 3; ++a) u_out[a * N + s] = double(uu[a]);
        if (Q_out)
#pragma unroll
            for (int k = 0; k < 5; ++k) Q_out[k * N + s] = double(Q[k * N + s]);
        v[0] = double(drho);
        if (Pi)
#pragma unroll
            for (int a = 0; a < 3; ++a) v[1 + a] = double(j[a]) + 0.5 * double(f[a]);
    }
    if (part) block_sum<4, BLK>(v, part + 4 * logical_block());
}

// Second stage: out[k] = sum_b part[b*stride + k], fixed order, one block.
__global__ __launch_bounds__(BLK) void k_reduce(const double *__restrict__ part, int nblk, int nv,
                                                int stride, double *__restrict__ out)
{
    __shared__ double buf[BLK];
    for (int k = 0; k < nv; ++k) {
        double s = 0.0;
        for (int b = threadIdx.x; b < nblk; b += BLK) s += part[b * stride + k];
        buf[threadIdx.x] = s;
        __syncthreads();
        for (int w = BLK / 2; w > 0; w >>= 1) {
            if (int(threadIdx.x) < w) buf[threadIdx.x] += buf[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[k] = buf[0];
        __syncthreads();
    }
}

// Local order q, director and disclination flag (q < threshold) per site;
// any output may be null.
template <typename T>
__global__ __launch_bounds__(BLK) void k_order(Geom G, const T *__restrict__ Q, double threshold,
                                               double *__restrict__ qo, double *__restrict__ dir,
                                               unsigned char *__restrict__ defect)
{
    const int s = site_index();
    if (s >= G.N) return;
    const size_t N = G.N;
    double q[5], lam, d[3];
#pragma unroll
    for (int k = 0; k < 5; ++k) q[k] = double(Q[k * N + s]);
    order_site(q, lam, d);
    if (qo) qo[s] = lam;
    if (dir)
#pragma unroll
        for (int a = 0; a < 3; ++a) dir[a * N + s] = d[a];
    if (defect) defect[s] = lam < threshold ? 1 : 0;
}

// Chunks of `len` sites that a plane is cut into for the per-plane sums: about 1024
// sites, more where that would take over 16 chunks.  Planes under 4096 sites stay
// whole where there are enough of them for the chip (`whole`): their chunks, of
// unequal size and an even number a plane, would all fall on the same XCDs.  f(z) of
// 64 x 20 x 1300 sites in two chunks a plane and in one: 46 and 40 us a call, in FP64
// 74 and 60; 512 x 6 x 512 43 and 38; 256 x 8 x 256 27 and 28; 64 x 64 x 512 in four and in
// one 38 and 40.  Counts: 64 x 20 x 1300 33 and 30, 512 x 6 x 512 29 and 31.
struct PlaneChunks {
    int len, n;
};

constexpr int FZ_WHOLE = 384, COUNT_WHOLE = 1024;

inline PlaneChunks plane_chunks(const Geom &G, int whole)
{
    const int sxy = G.nx * G.ny;
    const int most = sxy < 4096 && G.nz >= whole ? 1 : std::min(16, (sxy + 1023) / 1024);
    PlaneChunks c;
    c.len = ((sxy + most - 1) / most + BLK - 1) / BLK * BLK;
    c.n = (sxy + c.len - 1) / c.len;
    return c;
}

// Sums of the free-energy density over the chunks of a plane (block c + nc z),
// FP64, in a fixed order, so the profile f(z) is deterministic.  (One block per
// plane left the chip one wave per SIMD: 16.4 us on 64 x 64 x 256 sites, now 9.8.)
template <typename T>
__global__ __launch_bounds__(BLK) void k_fz(Geom G, Coef<T> c, const T *__restrict__ Q, PlaneChunks pc,
                                            double *__restrict__ part)
{
    const int z = blockIdx.x / pc.n, k0 = (blockIdx.x - z * pc.n) * pc.len;
    const int sxy = G.nx * G.ny, k1 = min(sxy, k0 + pc.len);
    double acc = 0.0;
    for (int k = k0 + int(threadIdx.x); k < k1; k += BLK) acc += double(fdens_at(G, c, Q, z * sxy + k));
    double v[1] = {acc};
    block_sum<1, BLK>(v, part + blockIdx.x);
}

// Disclination sites per chunk of a plane (block c + nc z), without the fields
// of the order analysis: the signs of three minors decide (order_below).  5.8
// us on 64 x 64 x 256 FP32 sites, where the eigen-solve per site, flags and a
// count over them took 63 + 7.5 us.
template <typename T>
__global__ __launch_bounds__(BLK) void k_count(Geom G, const T *__restrict__ Q, double threshold, PlaneChunks pc,
                                               int *__restrict__ cnt)
{
    __shared__ int total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const int z = blockIdx.x / pc.n, k0 = (blockIdx.x - z * pc.n) * pc.len;
    const int sxy = G.nx * G.ny, k1 = min(sxy, k0 + pc.len);
    const size_t N = G.N;
    int n = 0;
    for (int k = k0 + int(threadIdx.x); k < k1; k += BLK) {
        const size_t s = size_t(z) * sxy + k;
        double q[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) q[j] = double(Q[j * N + s]);
        n += order_below(q, threshold) ? 1 : 0;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) n += __shfl_down(n, w);
    if ((threadIdx.x & 63) == 0) atomicAdd(&total, n);
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = total;
}

// sin and cos by the library (one copy, out of the way of the registers of the
// kernel that needs it only for angles without a digit of phase).
__device__ __attribute__((noinline)) double2 sincos_far(double x)
{
    double s, c;
    sincos(x, &s, &c);
    return make_double2(s, c);
}

// sin and cos of x: the Taylor sums up to pi/4 (rest under 1e-19), beyond it
// after the nearest multiple of pi/2, in two parts, is taken off (rounded to
// 6e-17, up to 1e14); past that by the library.
__device__ __forceinline__ void sincos64(double x, double &sn, double &cs)
{
    int n = 0;
    if (!(fabs(x) <= 0.785)) {
        if (fabs(x) > 1e14) {
            const double2 f = sincos_far(x);
            sn = f.x;
            cs = f.y;
            return;
        }
        const double k = rint(x * 0.63661977236758134308);  // 2 / pi
        x = fma(-k, 6.12323399573676588614e-17, fma(-k, 1.57079632679489661923, x));
        n = int((long long)k & 3);
    }
    const double y = x * x;
    double s = 1.0 / 355687428096000.0, c = -1.0 / 6402373705728000.0;  // 1/17!, -1/18!
    constexpr double S[8] = {-1.0 / 1307674368000.0, 1.0 / 6227020800.0, -1.0 / 39916800.0, 1.0 / 362880.0,
                             -1.0 / 5040.0, 1.0 / 120.0, -1.0 / 6.0, 1.0};
    constexpr double C[9] = {1.0 / 20922789888000.0, -1.0 / 87178291200.0, 1.0 / 479001600.0, -1.0 / 3628800.0,
                             1.0 / 40320.0, -1.0 / 720.0, 1.0 / 24.0, -0.5, 1.0};
#pragma unroll
    for (int k = 0; k < 8; ++k) s = fma(s, y, S[k]);
#pragma unroll
    for (int k = 0; k < 9; ++k) c = fma(c, y, C[k]);
    s *= x;
    sn = n & 1 ? c : s;
    cs = n & 1 ? s : c;
    if (n & 2) sn = -sn;
    if (n == 1 || n == 2) cs = -cs;
}

// Polarised-light texture of the current Q (Sec. 2.3), the beam along +z
// (layer z = 0 first).  Unpolarised light behind the polariser at angle
// phi_in is S = (1, cos 2phi_in, sin 2phi_in, 0)/2; each site acts as a linear
// retarder with axis angle beta to x (cos 2beta = (dx^2 - dy^2)/(dx^2 + dy^2),
// sin 2beta = 2 dx dy/(dx^2 + dy^2)) and retardance
// delta = 2 pi q h / lambda (n_o n_e / sqrt(n_o^2 sin^2 alpha + n_e^2 cos^2 alpha) - n_o),
// cos alpha = d_z, from the FP64 local order q and director d (order_site).
// A retarder leaves S0 unchanged and turns (S1, S2, S3) by -delta about the axis
// (cos 2beta, sin 2beta, 0), kept as the quaternion (cos delta/2, -sin delta/2
// (cos 2beta, sin 2beta), 0): a layer costs 12 multiplications per wavelength
// (a 3x3 matrix 27).  The analyser at phi_out passes
// (S0 + cos 2phi_out S1 + sin 2phi_out S2)/2.
//
// A block holds 256 / SPB columns with their SPB z-segments, one thread each,
// for a group of up to OPT_G wavelengths: a thread multiplies the layers of its
// segment (later layers on the left), then one thread per column and
// wavelength the segments, out of LDS.  FP64 throughout.  Bound: the FP64
// arithmetic (630 instructions per site), two waves per SIMD for its registers:
// 50 us at 128^3, against 177 us with Jacobi sweeps and 3x3 matrices and 21 us
// for a second kernel that composed the segments.
constexpr int OPT_G = 3;

template <typename T, int SPB>
__global__ __launch_bounds__(BLK) void k_optics(Geom G, const T *__restrict__ Q, OpticsParams op, int wl0,
                                                double *__restrict__ image)
{
    constexpr int CPB = BLK / SPB;
    __shared__ double sq[SPB][OPT_G][4][CPB];
    __shared__ double so[OPT_G][CPB];
    const int cols = G.nx * G.ny;
    const int ci = threadIdx.x % CPB, seg = threadIdx.x / CPB, col = blockIdx.x * CPB + ci;
    const int ng = min(OPT_G, op.nwl - wl0);
    const int seglen = (G.nz + SPB - 1) / SPB;
    const int z0 = seg * seglen, z1 = col < cols ? min(G.nz, z0 + seglen) : 0;
    const size_t N = G.N;
    double w[OPT_G], x[OPT_G], y[OPT_G], zq[OPT_G], half[OPT_G];
#pragma unroll
    for (int g = 0; g < OPT_G; ++g) {
        w[g] = 1.0;
        x[g] = y[g] = zq[g] = 0.0;
        half[g] = g < ng ? fmin(0.5 / op.lam[wl0 + g], 1e308) : 0.0;  // finite: zero times it is zero
    }
    const double two_pi_h = 2.0 * 3.14159265358979323846 * op.h;
    const double no2 = op.n_o * op.n_o, ne2 = op.n_e * op.n_e, none = op.n_o * op.n_e;
#pragma unroll 1
    for (int z = z0; z < z1; ++z) {
        const size_t s = size_t(z) * cols + col;
        double q5[5], qo, d[3];
#pragma unroll
        for (int k = 0; k < 5; ++k) q5[k] = double(Q[k * N + s]);
        order_site(q5, qo, d);
        const double r2 = d[0] * d[0] + d[1] * d[1];
        double c = 1.0, sn = 0.0;
        // (closer to the beam the inverse overflows, and the retardance is zero to rounding about any axis)
        if (r2 > 1e-290) {
            const double ir2 = 1.0 / r2;
            c = (d[0] * d[0] - d[1] * d[1]) * ir2;
            sn = 2.0 * d[0] * d[1] * ir2;
        }
        const double cz = d[2] > 1.0 ? 1.0 : (d[2] < -1.0 ? -1.0 : d[2]);
        const double sin2a = 1.0 - cz * cz;
        const double base = two_pi_h * qo * (none * rsqrt64(no2 * sin2a + ne2 * cz * cz) - op.n_o);
#pragma unroll
        for (int g = 0; g < OPT_G; ++g) {
            if (g >= ng) break;
            double sd, w1;
            sincos64(base * half[g], sd, w1);
            const double x1 = -sd * c, y1 = -sd * sn;
            const double wn = w1 * w[g] - x1 * x[g] - y1 * y[g];
            const double xn = w1 * x[g] + x1 * w[g] + y1 * zq[g];
            const double yn = w1 * y[g] + y1 * w[g] - x1 * zq[g];
            zq[g] = w1 * zq[g] + x1 * y[g] - y1 * x[g];
            w[g] = wn;
            x[g] = xn;
            y[g] = yn;
        }
    }
#pragma unroll
    for (int g = 0; g < OPT_G; ++g) {
        sq[seg][g][0][ci] = w[g];
        sq[seg][g][1][ci] = x[g];
        sq[seg][g][2][ci] = y[g];
        sq[seg][g][3][ci] = zq[g];
    }
    __syncthreads();
    if (seg < ng) {  // thread (column ci, wavelength g = seg)
        const int g = seg, used = min(SPB, (G.nz + seglen - 1) / seglen);
        double a = 1.0, b = 0.0, c = 0.0, d = 0.0;
#pragma unroll 1
        for (int k = 0; k < used; ++k) {
            const double a1 = sq[k][g][0][ci], b1 = sq[k][g][1][ci], c1 = sq[k][g][2][ci], d1 = sq[k][g][3][ci];
            const double an = a1 * a - b1 * b - c1 * c - d1 * d;
            const double bn = a1 * b + b1 * a + c1 * d - d1 * c;
            const double cn = a1 * c - b1 * d + c1 * a + d1 * b;
            d = a1 * d + b1 * c - c1 * b + d1 * a;
            a = an;
            b = bn;
            c = cn;
        }
        const double n2 = a * a + b * b + c * c + d * d;  // 1 but for rounding
        const double v0 = ((a * a + b * b - c * c - d * d) * op.c_in + 2.0 * (b * c - a * d) * op.s_in) / n2;
        const double v1 = (2.0 * (b * c + a * d) * op.c_in + (a * a - b * b + c * c - d * d) * op.s_in) / n2;
        so[g][ci] = op.w[wl0 + g] * 0.25 * (1.0 + op.c_out * v0 + op.s_out * v1);
    }
    __syncthreads();
    if (seg != 0 || col >= cols) return;
    double out = 0.0;
    for (int g = 0; g < ng; ++g) out += so[g][ci];
    image[col] = wl0 == 0 ? out : image[col] + out;
}

// Disclination sites per z-plane: block z counts plane z (exact integer
// counts carried in FP64).
__global__ __launch_bounds__(BLK) void k_plane_count(Geom G, const unsigned char *__restrict__ defect,
                                                     double *__restrict__ cnt)
{
    const int z = blockIdx.x;
    const int sxy = G.nx * G.ny;
    double acc = 0.0;
    for (int k = threadIdx.x; k < sxy; k += BLK) acc += double(defect[size_t(z) * sxy + k]);
    double v[1] = {acc};
    block_sum<1, BLK>(v, cnt + z);
}

template <typename T>
__global__ __launch_bounds__(BLK) void k_fill(T *__restrict__ p, size_t n, T v)
{
    size_t i = size_t(blockIdx.x) * BLK + threadIdx.x;
    const size_t stride = size_t(gridDim.x) * BLK;
    for (; i < n; i += stride) p[i] = v;
}

// ---------------------------------------------------------------- launchers

inline int site_blocks(int N, int block = BLK) { return ((N + block - 1) / block + 7) / 8 * 8; }

// Records an event pair around each launch when a timer is attached.
struct Marks {
    KernelTimer *t;
    hipStream_t s;
    template <typename Fn>
    hipError_t operator()(int kind, Fn &&launch)
    {
        if (!t) {
            launch();
            return hipSuccess;
        }
        hipEvent_t a, b;
        hipError_t e = hipEventCreate(&a);
        if (e == hipSuccess) e = hipEventCreate(&b);
        if (e != hipSuccess) return e;
        (void)hipEventRecord(a, s);
        launch();
        (void)hipEventRecord(b, s);
        t->events.push_back({kind, a, b});
        return hipSuccess;
    }
};

int tile_tz(const Device &D) { return D.tz > 0 ? D.tz : 16; }
int tile_tzq(const Device &D) { return D.tzq > 0 ? D.tzq : tile_tz(D); }

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return cus;
}

// z-chunk for which the blocks of a tiled kernel fill the device's resident block
// slots `rounds` times: a launch of whole rounds leaves no CU idle at the end.
template <class S, class K>
int tz_fill_of(const Geom &G, K kernel, long long slots)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, S::NB, 0) != hipSuccess) return 0;
    return fill_chunk<S>(G.nx, G.ny, G.nz, slots * std::max(1, per_cu));
}

template <typename T, bool SPLIT>
int tz_fill_t(const Device &D, int kernel, int rounds)
{
    const Geom &G = D.G;
    const int cus = device_cus();
    if (cus < 1) return 0;
    const long long slots = (long long)cus * rounds;
    if (kernel == K_QUPDATE) return tz_fill_of<UpdateTile<T>>(G, k_qupdate<T>, slots);
    if (kernel == K_QFORCE) return tz_fill_of<KernelTile<T>>(G, k_qforce<T, false>, slots);
    if (kernel != K_QLB) return 0;
    // at 128^3 FP32 15 planes, 137 us a step where 16 take 138
    const int tz = tz_fill_of<WideTile<T>>(G, k_qlb<T, SPLIT, WideTile<T>>, slots);
    if (tz > 0 && wide_tiles<T>(G.nx, G.ny, G.nz, cus, tz)) return tz;
    return tz_fill_of<KernelTile<T>>(G, k_qlb<T, SPLIT, KernelTile<T>>, slots);
}

// Lattices whose per-site sweeps run in pairs over bricks: those of at most one
// brick per CU, which is as far as the doubled evaluations stay hidden behind
// the two launches saved.  A step in us, single sweeps and pairs: 16^3 (32 bricks)
// 13.7 and 9.3 in FP32, 17.0 and 12.1 in FP64; 32^3 (256) 13.3 and 9.3, 17.8 and
// 13.2; past one brick per CU 64 x 32 x 32 (512) 13.3 and 12.5, but 19.2 and 20.2
// in FP64; 40^3 (600) 14.2 and 17.2, 19.7 and 25.8; 64^3 (2048) 26 and 32, 50 and
// 65.  The brick: larger ones (8 x 8 x 4, 16 x 8 x 4) evaluate fewer face points,
// but leave CUs idle on the lattices in question.
// One limit for both pairs and precisions, below which all gain.
typedef Brick<16, 4, 2> StepBrick;

bool small_lattice(const Geom &G, int cus) { return StepBrick::blocks(G) <= cus; }

// Threads per block of the per-site sweeps of a step.  With few blocks of 256
// some CUs get one more than others and the launch waits for them, so where
// that is more than a tenth, up to five blocks a CU, a block is one wave.  A
// step in us with 256 and 64: 44^3 (333 blocks on 256 CUs) 19.4 and 18.7 in
// FP32, 28.5 and 25.8 in FP64; 60 x 44 x 53 (547) 23.2 and 22.0, 38.3 and 33.2;
// 70 x 66 x 61 (1101) 31.8 and 31.5, 59.5 and 57.5.  Even, 64^3 (1024): 26.8 and
// 27.5, 51.0 and 50.0.  More blocks: 96 x 80 x 70 (2100) 45.5 and 47.4, 95.8 and
// 95.7; 128^3 (8192) 139 and 150, 336 and 349.
template <class F>
void with_block(int N, int cus, F &&f)
{
    const int nb = site_blocks(N), rounds = (nb + cus - 1) / std::max(1, cus);
    if (rounds <= 5 && 10 * (rounds * cus - nb) > nb) f(std::integral_constant<int, 64>{});
    else f(std::integral_constant<int, BLK>{});
}
// Launches a per-site kernel template over the sites of the lattice, B threads per block.
#define SWEEP_OF(N, KERNEL, ...)                                                  \
    with_block(N, cus, [&](auto block) {                                          \
        constexpr int B = decltype(block)::value;                                 \
        KERNEL<<<site_blocks(N, B), B, 0, D.stream>>>(__VA_ARGS__);               \
    })
#define SWEEP(KERNEL, ...) SWEEP_OF(G.N, KERNEL, __VA_ARGS__)

template <typename T, bool SPLIT>
hipError_t steps_t(Device &D, const PhysParams &p, int nsteps, KernelTimer *timer)
{
    const bool pc = p.model == LB_D3Q15_PC;
    const int sc = D.sched;
    // the tiled stress kernels run the D3Q19 LB only, and k_qforce the whole stress only
    const bool tiled_stress = sc == SCHED_TILED || sc == SCHED_FUSED || sc == SCHED_FUSED_TILED;
    if ((pc && tiled_stress) || (SPLIT && sc == SCHED_TILED)) return hipErrorNotSupported;
    // the Q update: tiled predictor-corrector, or the per-site predictor and corrector
    const bool tiled_q = sc == SCHED_TILED || sc == SCHED_MIXED || sc == SCHED_FUSED_TILED;
    const bool dbg_nan = (D.debug & DEBUG_NAN_LDS) != 0;
    const Geom G = D.G;
    const Coef<T> c = make_coef<T>(p);
    const int cus = device_cus();
    T *u = static_cast<T *>(D.u), *Pi = static_cast<T *>(D.Pi);
    Marks mark{timer, D.stream};
    hipError_t e = hipSuccess;
    if (!p.flow && nsteps > 0)  // pure relaxation: u == 0 (Sec. 2.1)
        k_fill<T><<<1024, BLK, 0, D.stream>>>(u, 3 * size_t(G.N), T(0));
    const TileGrid tg = tile_grid(G.nx, G.ny, G.nz, KernelTile<T>::TX, KernelTile<T>::TY, tile_tz(D));
    const TileGrid tgq = tile_grid(G.nx, G.ny, G.nz, UpdateTile<T>::TX, UpdateTile<T>::TY, tile_tzq(D));
    const TileGrid tgw = tile_grid(G.nx, G.ny, G.nz, WideTile<T>::TX, WideTile<T>::TY, tile_tz(D));
    const bool wide = wide_tiles<T>(G.nx, G.ny, G.nz, cus, std::min(G.nz, tile_tz(D)));
    const int tzp = pc ? pass_chunk<T>(G.nx, G.ny, G.nz, cus, SPLIT) : 0;
    const int tb = KernelTile<T>::NB;
    const bool pairs = sc == SCHED_SITES && small_lattice(G, cus);
    const int nbr = StepBrick::blocks(G), lbr = (nbr + 7) / 8 * 8;
    for (int n = 0; n < nsteps && e == hipSuccess; ++n) {
        T *Q = static_cast<T *>(D.Q[D.qcur]);
        T *Qs = static_cast<T *>(D.Q[D.qcur ^ 1]);  // predictor stage, or Q^{n+1} of the tiled update
        if (p.flow) {
            T *gin = static_cast<T *>(D.g[D.gcur]);
            T *gout = static_cast<T *>(D.g[D.gcur ^ 1]);
            if (sc == SCHED_FUSED || sc == SCHED_FUSED_TILED) {
                e = mark(K_QLB, [&] {
                    if (wide)
                        k_qlb<T, SPLIT, WideTile<T>><<<tgw.launch, WideTile<T>::NB, 0, D.stream>>>(G, c, tgw, Q, gin,
                                                                                                   gout, u, dbg_nan);
                    else
                        k_qlb<T, SPLIT, KernelTile<T>><<<tg.launch, tb, 0, D.stream>>>(G, c, tg, Q, gin, gout, u,
                                                                                       dbg_nan);
                });
            } else if (sc == SCHED_TILED) {
                e = mark(K_QFORCE, [&] {
                    k_qforce<T, false><<<tg.launch, tb, 0, D.stream>>>(G, c, tg, Q, Pi, nullptr, dbg_nan);
                });
                if (e == hipSuccess)
                    e = mark(K_LBF, [&] { k_lbf<T><<<site_blocks(G.N), BLK, 0, D.stream>>>(G, c, gin, Pi, gout, u); });
            } else if (pairs && !pc) {
                e = mark(K_QLB, [&] {
                    k_blb<T, SPLIT, StepBrick><<<lbr, StepBrick::NB, 0, D.stream>>>(G, c, nbr, Q, gin, gout, u);
                });
            } else {
                e = mark(K_STRESS, [&] { SWEEP((k_stress<T, SPLIT, B>), G, c, Q, Pi, nullptr); });
                if (pc && tzp) {
                    const TileGrid tp = tile_grid(G.nx, G.ny, G.nz, PassTile<T>::TX, PassTile<T>::TY, tzp);
                    if (e == hipSuccess)
                        e = mark(K_PC2, [&] {
                            k_pc<T, SPLIT><<<tp.launch, PassTile<T>::NB, 0, D.stream>>>(G, c, tp, gin, Pi, gout, u);
                        });
                } else if (pc) {
                    T *P = static_cast<T *>(D.aux);
                    T *bsave = gout + 15 * size_t(G.N);  // planes 15..17 of the target buffer
                    if (e == hipSuccess)
                        e = mark(K_PC1, [&] {
                            SWEEP((k_pc1<T, SPLIT, B>), G, c, gin, Pi, P, u, bsave);
                        });
                    if (e == hipSuccess)
                        e = mark(K_PC2, [&] {
                            SWEEP((k_pc2<T, SPLIT, B>), G, c, gin, P, Pi, bsave, gout);
                        });
                } else if (e == hipSuccess) {
                    e = mark(K_LB, [&] { SWEEP((k_lb<T, SPLIT, B>), G, c, gin, Pi, gout, u); });
                }
            }
            D.gcur ^= 1;
        }
        if (tiled_q) {
            if (e == hipSuccess)
                e = mark(K_QUPDATE, [&] {
                    k_qupdate<T><<<tgq.launch, UpdateTile<T>::NB, 0, D.stream>>>(G, c, tgq, Q, u, Qs, dbg_nan);
                });
            D.qcur ^= 1;
        } else if (pairs && (p.flow || (n ^ 1) < nsteps)) {
            // without flow only Q alternates: the last of an odd number of steps goes by the
            // in-place sweeps below, so that a caller's graph of any such call can be replayed
            if (e == hipSuccess)
                e = mark(K_QUPDATE,
                         [&] { k_bq<T, StepBrick><<<lbr, StepBrick::NB, 0, D.stream>>>(G, c, nbr, Q, u, Qs); });
            D.qcur ^= 1;
        } else if (sizeof(T) == 8 && G.nx % 2 == 0) {
            if constexpr (sizeof(T) == 8) {
                if (e == hipSuccess)
                    e = mark(K_QPRED, [&] { SWEEP_OF(G.N / 2, (k_qpred2<T, B>), G, c, Q, u, Qs); });
                if (e == hipSuccess)
                    e = mark(K_QCORR, [&] { SWEEP_OF(G.N / 2, (k_qcorr2<T, B>), G, c, Q, Qs, u); });
            }
        } else {
            if (e == hipSuccess)
                e = mark(K_QPRED, [&] { SWEEP((k_qpred<T, B>), G, c, Q, u, Qs); });
            if (e == hipSuccess)
                e = mark(K_QCORR, [&] { SWEEP((k_qcorr<T, B>), G, c, Q, Qs, u); });
        }
    }
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

template <typename T>
hipError_t init_t(Device &D, const PhysParams &p, const double *stage)
{
    const Geom G = D.G;
    const Coef<T> c = make_coef<T>(p);
    const size_t N = G.N;
    const int nb = site_blocks(G.N);
    if (p.model == LB_D3Q15_PC)
        k_init15<T><<<nb, BLK, 0, D.stream>>>(G, c, stage, stage + N, stage + 4 * N,
                                              static_cast<T *>(D.g[D.gcur]), static_cast<T *>(D.Q[D.qcur]));
    else
        k_init<T><<<nb, BLK, 0, D.stream>>>(G, c, stage, stage + N, stage + 4 * N,
                                            static_cast<T *>(D.g[D.gcur]), static_cast<T *>(D.Q[D.qcur]));
    // u of the last LB step: zero until the first step (and for good with flow off)
    k_fill<T><<<1024, BLK, 0, D.stream>>>(static_cast<T *>(D.u), 3 * N, T(0));
    return hipGetLastError();
}

template <typename T, bool SPLIT>
hipError_t readout_t(Device &D, const PhysParams &p, double *stage, double *totals, double *part)
{
    const Geom G = D.G;
    const Coef<T> c = make_coef<T>(p);
    const size_t N = G.N;
    const int nb = site_blocks(G.N);
    T *Pi = static_cast<T *>(D.Pi);
    const T *Q = static_cast<const T *>(D.Q[D.qcur]);
    if (p.model == LB_D3Q15_PC) {
        // the stress sweep only for the free-energy partials
        if (totals) k_stress<T, SPLIT><<<nb, BLK, 0, D.stream>>>(G, c, Q, Pi, part + 4 * nb);
        k_readout15<T><<<nb, BLK, 0, D.stream>>>(G, c, static_cast<const T *>(D.g[D.gcur]), p.flow != 0, Q, stage,
                                                 stage ? stage + N : nullptr, stage ? stage + 4 * N : nullptr,
                                                 totals ? part : nullptr);
        if (totals) {
            k_reduce<<<1, BLK, 0, D.stream>>>(part, nb, 4, 4, totals);
            k_reduce<<<1, BLK, 0, D.stream>>>(part + 4 * nb, nb, 1, 1, totals + 4);
        }
        return hipGetLastError();
    }
    if (totals)
        k_stress<T, SPLIT><<<nb, BLK, 0, D.stream>>>(G, c, Q, Pi, part + 4 * nb);
    else if (p.flow)
        k_stress<T, SPLIT><<<nb, BLK, 0, D.stream>>>(G, c, Q, Pi, nullptr);
    k_readout<T, SPLIT><<<nb, BLK, 0, D.stream>>>(G, c, static_cast<const T *>(D.g[D.gcur]), p.flow ? Pi : nullptr,
                                                  Q, stage, stage ? stage + N : nullptr,
                                                  stage ? stage + 4 * N : nullptr, totals ? part : nullptr);
    if (totals) {
        k_reduce<<<1, BLK, 0, D.stream>>>(part, nb, 4, 4, totals);
        k_reduce<<<1, BLK, 0, D.stream>>>(part + 4 * nb, nb, 1, 1, totals + 4);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t fz_t(Device &D, const PhysParams &p, double *part)
{
    const PlaneChunks pc = plane_chunks(D.G, FZ_WHOLE);
    k_fz<T><<<D.G.nz * pc.n, BLK, 0, D.stream>>>(D.G, make_coef<T>(p), static_cast<const T *>(D.Q[D.qcur]), pc, part);
    return hipGetLastError();
}

template <typename T>
void optics_t(Device &D, const OpticsParams &op, double *image)
{
    const int cols = D.G.nx * D.G.ny;
    const T *Q = static_cast<const T *>(D.Q[D.qcur]);
    for (int wl0 = 0; wl0 < op.nwl; wl0 += OPT_G) {
        // 16 segments where the columns alone give the chip some 500 blocks, 64 below
        if (cols >= 8192)
            k_optics<T, 16><<<(cols + 15) / 16, BLK, 0, D.stream>>>(D.G, Q, op, wl0, image);
        else
            k_optics<T, 64><<<(cols + 3) / 4, BLK, 0, D.stream>>>(D.G, Q, op, wl0, image);
    }
}

}  // namespace

hipError_t run_order(Device &D, double threshold, double *q, double *dir, unsigned char *defect, double *cnt)
{
    const int nb = site_blocks(D.G.N);
    if (D.fp32)
        k_order<float><<<nb, BLK, 0, D.stream>>>(D.G, static_cast<const float *>(D.Q[D.qcur]), threshold, q, dir,
                                                 defect);
    else
        k_order<double><<<nb, BLK, 0, D.stream>>>(D.G, static_cast<const double *>(D.Q[D.qcur]), threshold, q,
                                                  dir, defect);
    if (cnt) k_plane_count<<<D.G.nz, BLK, 0, D.stream>>>(D.G, defect, cnt);
    return hipGetLastError();
}

int fz_parts(const Geom &G) { return plane_chunks(G, FZ_WHOLE).n; }
int count_parts(const Geom &G) { return plane_chunks(G, COUNT_WHOLE).n; }

hipError_t run_count(Device &D, double threshold, int *cnt)
{
    const PlaneChunks pc = plane_chunks(D.G, COUNT_WHOLE);
    if (D.fp32)
        k_count<float><<<D.G.nz * pc.n, BLK, 0, D.stream>>>(D.G, static_cast<const float *>(D.Q[D.qcur]), threshold,
                                                            pc, cnt);
    else
        k_count<double><<<D.G.nz * pc.n, BLK, 0, D.stream>>>(D.G, static_cast<const double *>(D.Q[D.qcur]), threshold,
                                                             pc, cnt);
    return hipGetLastError();
}

hipError_t run_optics(Device &D, const OpticsParams &op, double *image)
{
    if (D.fp32)
        optics_t<float>(D, op, image);
    else
        optics_t<double>(D, op, image);
    return hipGetLastError();
}

hipError_t run_fz(Device &D, const PhysParams &p, double *part)
{
    return D.fp32 ? fz_t<float>(D, p, part) : fz_t<double>(D, p, part);
}

size_t partial_doubles(int nx, int ny, int nz)
{
    // per-site blocks x 4 (readout moments) + per-site blocks (free energy),
    // or the chunks of every z-plane (free-energy profile; at most one per 1024
    // sites and one more a plane)
    return size_t(5) * site_blocks(nx * ny * nz) + size_t(nz) + 16;
}

const char *kernel_name(int k)
{
    static const char *names[K_COUNT] = {"k_stress", "k_lb", "k_qpred", "k_qcorr", "k_qforce", "k_lbf",
                                         "k_qupdate", "k_pc1", "k_pc2", "k_qlb"};
    return (k >= 0 && k < K_COUNT) ? names[k] : nullptr;
}

hipError_t run_steps(Device &D, const PhysParams &p, int nsteps, KernelTimer *timer)
{
    if (p.flow == FLOW_SPLIT)
        return D.fp32 ? steps_t<float, true>(D, p, nsteps, timer) : steps_t<double, true>(D, p, nsteps, timer);
    return D.fp32 ? steps_t<float, false>(D, p, nsteps, timer) : steps_t<double, false>(D, p, nsteps, timer);
}

int tile_tz_fill(const Device &D, int kernel, bool split, int rounds)
{
    if (split) return D.fp32 ? tz_fill_t<float, true>(D, kernel, rounds) : tz_fill_t<double, true>(D, kernel, rounds);
    return D.fp32 ? tz_fill_t<float, false>(D, kernel, rounds) : tz_fill_t<double, false>(D, kernel, rounds);
}

hipError_t run_init(Device &D, const PhysParams &p, const double *stage)
{
    return D.fp32 ? init_t<float>(D, p, stage) : init_t<double>(D, p, stage);
}

hipError_t run_readout(Device &D, const PhysParams &p, double *stage, double *totals, double *part)
{
    if (!part) part = D.part;
    if (p.flow == FLOW_SPLIT)
        return D.fp32 ? readout_t<float, true>(D, p, stage, totals, part)
                      : readout_t<double, true>(D, p, stage, totals, part);
    return D.fp32 ? readout_t<float, false>(D, p, stage, totals, part)
                  : readout_t<double, false>(D, p, stage, totals, part);
}

size_t readout_partials(const Geom &G) { return size_t(5) * site_blocks(G.N); }

}  // namespace hlb
