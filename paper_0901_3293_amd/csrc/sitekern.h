// sitekern.h -- one-site-per-thread work of the step, as device functions
// over a linear site index of one periodic box.  The plain kernels and the
// batched kernels all call these; neighbour values come straight from global
// memory through the L1/L2 of the executing CU.  A site index is split into
// (x, y, z) by multiply-high division (FastDiv in kernels.h), and every field
// plane is read through its wave-uniform base address plus 32-bit byte
// offsets (Off below).
//
// Buffers of one box (structure-of-arrays, component stride N, x fastest):
//   g 19 x N, Q 5 x N, Qs (predictor stage) 5 x N, u 3 x N, Pi 9 x N
//   (whole-stress coupling) or 12 x N (split coupling: sigma^xi xx, xy, xz,
//   yy, yz, zz; tau xy, xz, yz; h x, y, z).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "site.h"

namespace hlb {

struct Nbr {
    int s, x, y, z;
    int nb[6];  // x+1, x-1, y+1, y-1, z+1, z-1 (periodic)
};

// The site s = x + nx (y + ny z) at (x, y, z) and its six periodic neighbours.
__device__ __forceinline__ Nbr nbr_at(const Geom &G, int s, int x, int y, int z)
{
    Nbr S;
    const int sxy = G.nx * G.ny;
    S.s = s;
    S.x = x;
    S.y = y;
    S.z = z;
    S.nb[0] = (x == G.nx - 1) ? s - (G.nx - 1) : s + 1;
    S.nb[1] = (x == 0) ? s + (G.nx - 1) : s - 1;
    S.nb[2] = (y == G.ny - 1) ? s - G.nx * (G.ny - 1) : s + G.nx;
    S.nb[3] = (y == 0) ? s + G.nx * (G.ny - 1) : s - G.nx;
    S.nb[4] = (z == G.nz - 1) ? s - sxy * (G.nz - 1) : s + sxy;
    S.nb[5] = (z == 0) ? s + sxy * (G.nz - 1) : s - sxy;
    return S;
}

// The same from the linear site index.
__device__ __forceinline__ Nbr nbr_of(const Geom &G, int s)
{
    const int yz = int(fastdiv(unsigned(s), G.dx));
    const int z = int(fastdiv(unsigned(yz), G.dy));
    return nbr_at(G, s, s - yz * G.nx, yz - z * G.ny, z);
}

// Byte offsets of a site and of its six neighbours within one field plane of
// elements of type T.  A plane of N values is under 4 GiB (checked when a
// context is created), so 32-bit offsets from the plane's base address it;
// the base (field + c N) is the same for the whole wave, and one site's
// offsets serve every component of every field.
template <typename T>
struct Off {
    unsigned s;
    unsigned nb[6];  // x+1, x-1, y+1, y-1, z+1, z-1
};

template <typename T>
__device__ __forceinline__ Off<T> offsets(const Nbr &S)
{
    Off<T> O;
    O.s = unsigned(S.s) * unsigned(sizeof(T));
#pragma unroll
    for (int k = 0; k < 6; ++k) O.nb[k] = unsigned(S.nb[k]) * unsigned(sizeof(T));
    return O;
}

// Plane c of a component-major field of N values per component.
template <typename T>
__device__ __forceinline__ T *plane(T *f, int c, int N)
{
    return f + size_t(c) * size_t(N);
}

template <typename T>
__device__ __forceinline__ T *at(T *P, unsigned b)
{
    return reinterpret_cast<T *>(reinterpret_cast<char *>(P) + b);
}

template <typename T>
__device__ __forceinline__ const T *at(const T *P, unsigned b)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(P) + b);
}

// Byte offset of the site x - e of a population with velocity e = (cx, cy,
// cz): each nonzero component adds the byte distance to the neighbour on the
// opposite side (periodic), so a pull costs one or two additions.
template <typename T>
__device__ __forceinline__ unsigned pull_off(const Off<T> &O, int cx, int cy, int cz)
{
    unsigned b = O.s;
    if (cx > 0) b += O.nb[1] - O.s;
    else if (cx < 0) b += O.nb[0] - O.s;
    if (cy > 0) b += O.nb[3] - O.s;
    else if (cy < 0) b += O.nb[2] - O.s;
    if (cz > 0) b += O.nb[5] - O.s;
    else if (cz < 0) b += O.nb[4] - O.s;
    return b;
}

// Population access.  In a sweep over one whole box every population value
// is read once and written once per step, and the next reader of the written
// value is the next step's sweep, after the Q-side kernels have moved their
// own fields; with STREAM the loads and stores are nontemporal so that the
// populations do not push Q, u and the stress out of the L2 and the
// last-level cache between the kernels of a step.  (The predicted
// populations of the first D3Q15 pass are read once, by the second pass right
// after it, but at 15 values per site they are too many to stay cached beside
// the rest: they are streamed too.)  The batched kernels stream them as
// well, so that a cache group's other fields stay in the last-level cache.
template <bool STREAM, typename T>
__device__ __forceinline__ T pop_load(const T *P, unsigned b)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(at(P, b));
    else return *at(P, b);
}

template <bool STREAM, typename T>
__device__ __forceinline__ void pop_store(T *P, unsigned b, T v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, at(P, b));
    else *at(P, b) = v;
}

// Pulled source of population i arriving at (x,y,z): site (x,y,z) - e_i.
__device__ __forceinline__ int pull_from(const Geom &G, const Nbr &S, int cx, int cy, int cz)
{
    int xs = S.x - cx, ys = S.y - cy, zs = S.z - cz;
    xs += (xs < 0) ? G.nx : ((xs >= G.nx) ? -G.nx : 0);
    ys += (ys < 0) ? G.ny : ((ys >= G.ny) ? -G.ny : 0);
    zs += (zs < 0) ? G.nz : ((zs >= G.nz) ? -G.nz : 0);
    return xs + G.nx * (ys + G.ny * zs);
}

// Centred derivatives and 7-point Laplacian of a value from its neighbours.
template <typename T>
__device__ __forceinline__ void stencil7(T v, T xp, T xm, T yp, T ym, T zp, T zm, T &dx, T &dy, T &dz, T &lap)
{
    dx = T(0.5) * (xp - xm);
    dy = T(0.5) * (yp - ym);
    dz = T(0.5) * (zp - zm);
    lap = ((xp + xm) + (yp + ym)) + (zp + zm) - T(6) * v;
}

// Derivatives of the 5-component Q at one site.
template <typename T>
__device__ __forceinline__ void gather_q(const T *__restrict__ Q, int N, const Off<T> &O, T q[5], T d[3][5],
                                         T lap[5])
{
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const T *P = plane(Q, c, N);
        q[c] = *at(P, O.s);
        stencil7(q[c], *at(P, O.nb[0]), *at(P, O.nb[1]), *at(P, O.nb[2]), *at(P, O.nb[3]), *at(P, O.nb[4]),
                 *at(P, O.nb[5]), d[0][c], d[1][c], d[2][c], lap[c]);
    }
}

template <typename T>
__device__ __forceinline__ void gather_u(const T *__restrict__ u, int N, const Off<T> &O, T uc[3], T W[3][3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T *P = plane(u, a, N);
        uc[a] = *at(P, O.s);
        W[a][0] = T(0.5) * (*at(P, O.nb[0]) - *at(P, O.nb[1]));
        W[a][1] = T(0.5) * (*at(P, O.nb[2]) - *at(P, O.nb[3]));
        W[a][2] = T(0.5) * (*at(P, O.nb[4]) - *at(P, O.nb[5]));
    }
}

// Body force F_a = sum_b [Pi_ab(x + e_b) - Pi_ab(x - e_b)] / 2 (Eq. (19)).
template <typename T>
__device__ __forceinline__ void divergence(const T *__restrict__ Pi, int N, const Off<T> &O, T F[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T *Px = plane(Pi, 3 * a + 0, N);
        const T *Py = plane(Pi, 3 * a + 1, N);
        const T *Pz = plane(Pi, 3 * a + 2, N);
        F[a] = T(0.5) * ((*at(Px, O.nb[0]) - *at(Px, O.nb[1])) + (*at(Py, O.nb[2]) - *at(Py, O.nb[3])) +
                         (*at(Pz, O.nb[4]) - *at(Pz, O.nb[5])));
    }
}

// Stress Pi(Q) at one site (Eqs. (6)-(8)); returns the free-energy density.
template <typename T>
__device__ __forceinline__ T stress_at(const Geom &G, const Coef<T> &c, const T *__restrict__ Q,
                                       T *__restrict__ Pi, int s)
{
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T q[5], d[3][5], lap[5], P[3][3], fd, H[5];
    gather_q(Q, G.N, O, q, d, lap);
    site_stress(c, q, d, lap, P, fd, H);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) *at(plane(Pi, 3 * a + b, G.N), O.s) = P[a][b];
    return fd;
}

// Pull-stream, BGK collision with the body force div Pi (Eqs. (14), (16),
// (19)) at one site; writes g' and u.
template <typename T, bool STREAM = false>
__device__ __forceinline__ void lb_at(const Geom &G, const Coef<T> &c, const T *__restrict__ gin,
                                      const T *__restrict__ Pi, T *__restrict__ gout, T *__restrict__ u, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T g[19], F[3], uu[3], rho;
#pragma unroll
    for (int i = 0; i < 19; ++i) g[i] = pop_load<STREAM>(plane(gin, i, N), pull_off(O, CX[i], CY[i], CZ[i]));
    divergence(Pi, N, O, F);
    lb_collide(c, g, F, uu, rho);
#pragma unroll
    for (int i = 0; i < 19; ++i) pop_store<STREAM>(plane(gout, i, N), O.s, g[i]);
#pragma unroll
    for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
}

// Split-coupling terms at one site (planes of the 12 x N layout above);
// returns the free-energy density.
template <typename T>
__device__ __forceinline__ T split_at(const Geom &G, const Coef<T> &c, const T *__restrict__ Q, T *__restrict__ P,
                                      int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T q[5], d[3][5], lap[5], sig[6], tau3[3], h[3], fd;
    gather_q(Q, N, O, q, d, lap);
    site_split(c, q, d, lap, sig, tau3, h, fd);
#pragma unroll
    for (int k = 0; k < 6; ++k) *at(plane(P, k, N), O.s) = sig[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) *at(plane(P, 6 + k, N), O.s) = tau3[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) *at(plane(P, 9 + k, N), O.s) = h[k];
    return fd;
}

// Split body force b_a = d_b tau_ab + h_a (centred on the second index;
// tau antisymmetric, stored as xy, xz, yz).
template <typename T>
__device__ __forceinline__ void split_force(const T *__restrict__ P, int N, const Off<T> &O, T b[3])
{
    const T *txy = plane(P, 6, N), *txz = plane(P, 7, N), *tyz = plane(P, 8, N);
    b[0] = T(0.5) * ((*at(txy, O.nb[2]) - *at(txy, O.nb[3])) + (*at(txz, O.nb[4]) - *at(txz, O.nb[5]))) +
           *at(plane(P, 9, N), O.s);
    b[1] = T(0.5) * ((*at(tyz, O.nb[4]) - *at(tyz, O.nb[5])) - (*at(txy, O.nb[0]) - *at(txy, O.nb[1]))) +
           *at(plane(P, 10, N), O.s);
    b[2] = T(0.5) * (-(*at(txz, O.nb[0]) - *at(txz, O.nb[1])) - (*at(tyz, O.nb[2]) - *at(tyz, O.nb[3]))) +
           *at(plane(P, 11, N), O.s);
}

// LB step of the split coupling at one site: pull, collide with the stress in
// the equilibrium and the split body force; writes g' and u.
template <typename T, bool STREAM = false>
__device__ __forceinline__ void lb_split_at(const Geom &G, const Coef<T> &c, const T *__restrict__ gin,
                                            const T *__restrict__ P, T *__restrict__ gout, T *__restrict__ u, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T g[19], b[3], sig[6], uu[3], rho;
#pragma unroll
    for (int i = 0; i < 19; ++i) g[i] = pop_load<STREAM>(plane(gin, i, N), pull_off(O, CX[i], CY[i], CZ[i]));
    split_force(P, N, O, b);
#pragma unroll
    for (int k = 0; k < 6; ++k) sig[k] = *at(plane(P, k, N), O.s);
    lb_collide_split(c, g, b, sig, uu, rho);
#pragma unroll
    for (int i = 0; i < 19; ++i) pop_store<STREAM>(plane(gout, i, N), O.s, g[i]);
#pragma unroll
    for (int a = 0; a < 3; ++a) *at(plane(u, a, N), O.s) = uu[a];
}

// Body force b = div Pi of the D3Q15 LB at one site, or SPLIT b = div tau + h
// beside sigma^xi.
template <typename T, bool SPLIT>
__device__ __forceinline__ void force15(const T *__restrict__ Pi, int N, const Off<T> &O, T b[3], T sig[6])
{
    if constexpr (SPLIT) {
        split_force(Pi, N, O, b);
#pragma unroll
        for (int k = 0; k < 6; ++k) sig[k] = *at(plane(Pi, k, N), O.s);
    } else {
        divergence(Pi, N, O, b);
    }
}

// D3Q15 predictor-corrector LB (Eq. (15)), first pass at one site x: the
// collision C(x, {f}) of the local populations with the stress and body force
// of this step (split: sigma^xi from the 12-plane layout and b = div tau + h;
// whole-stress coupling: no stress term and b = div Pi); writes the
// predictor populations P = f + C at x (to be streamed), the velocity u^n of
// f(x, t) and b (3 planes, read back by the second pass at the same site).
template <typename T, bool SPLIT, bool STREAM = false>
__device__ __forceinline__ void pc1_at(const Geom &G, const Coef<T> &c, const T *__restrict__ g,
                                       const T *__restrict__ Pi, T *__restrict__ P, T *__restrict__ u,
                                       T *__restrict__ bsave, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T f[15], C[15], b[3], sig[6], uu[3], rho;
#pragma unroll
    for (int i = 0; i < 15; ++i) f[i] = *at(plane(g, i, N), O.s);
    force15<T, SPLIT>(Pi, N, O, b, sig);
    lb15_collide<T, SPLIT>(c, f, sig, b, C, uu, rho);
#pragma unroll
    for (int i = 0; i < 15; ++i) pop_store<STREAM>(plane(P, i, N), O.s, f[i] + C[i]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        *at(plane(u, a, N), O.s) = uu[a];
        *at(plane(bsave, a, N), O.s) = b[a];
    }
}

// Second pass at one site y: f*_i(y) = P_i(y - e_i), collision C(y, {f*}),
//   f_i(y, t + 1) = [f_i(y - e_i) + P_i(y - e_i)]/2 + C_i(y, {f*})/2.
template <typename T, bool SPLIT, bool STREAM = false>
__device__ __forceinline__ void pc2_at(const Geom &G, const Coef<T> &c, const T *__restrict__ g,
                                       const T *__restrict__ P, const T *__restrict__ Pi,
                                       const T *__restrict__ bsave, T *__restrict__ gout, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T fs[15], fo[15], C[15], b[3], sig[6], uu[3], rho;
#pragma unroll
    for (int i = 0; i < 15; ++i) {
        const unsigned t = pull_off(O, DX15[i], DY15[i], DZ15[i]);
        fs[i] = pop_load<STREAM>(plane(P, i, N), t);
        fo[i] = T(0.5) * (pop_load<STREAM>(plane(g, i, N), t) + fs[i]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) b[a] = *at(plane(bsave, a, N), O.s);
    if (SPLIT)
#pragma unroll
        for (int k = 0; k < 6; ++k) sig[k] = *at(plane(Pi, k, N), O.s);
    lb15_collide<T, SPLIT>(c, fs, sig, b, C, uu, rho);
#pragma unroll
    for (int i = 0; i < 15; ++i) pop_store<STREAM>(plane(gout, i, N), O.s, fmat(T(0.5), C[i], fo[i]));
}

// Predictor Q* = Q + R(Q, u) at one site (Eqs. (2)-(4)).
template <typename T>
__device__ __forceinline__ void pred_at(const Geom &G, const Coef<T> &c, const T *__restrict__ Q,
                                        const T *__restrict__ u, T *__restrict__ Qs, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T q[5], d[3][5], lap[5], uc[3], W[3][3], R[5];
    gather_q(Q, N, O, q, d, lap);
    gather_u(u, N, O, uc, W);
    site_rhs(c, q, d, lap, uc, W, R);
#pragma unroll
    for (int k = 0; k < 5; ++k) *at(plane(Qs, k, N), O.s) = q[k] + R[k];
}

// Corrector Q^{n+1} = Q^n + [R(Q^n) + R(Q*)]/2 = [Q^n + Q* + R(Q*)]/2, in
// place over Q (each site reads only its own Q^n).
template <typename T>
__device__ __forceinline__ void corr_at(const Geom &G, const Coef<T> &c, T *__restrict__ Q,
                                        const T *__restrict__ Qs, const T *__restrict__ u, int s)
{
    const int N = G.N;
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T qn[5], q[5], d[3][5], lap[5], uc[3], W[3][3], R[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) qn[k] = *at(plane(Q, k, N), O.s);  // issued with the stencil loads
    gather_q(Qs, N, O, q, d, lap);
    gather_u(u, N, O, uc, W);
    site_rhs(c, q, d, lap, uc, W, R);
#pragma unroll
    for (int k = 0; k < 5; ++k) *at(plane(Q, k, N), O.s) = T(0.5) * (qn[k] + q[k] + R[k]);
}

// ---- two sites per thread: (x, x + 1), x even, nx even.  The rows are read two
// values at a time; the neighbours in x are the thread's own other site and the
// sites of the lanes below and above, or a load at the ends of a row or a wave.
// All lanes of a wave take part (one past the last pair repeats it).
template <typename T>
using Two = T __attribute__((ext_vector_type(2)));

template <typename T>
struct PairAt {
    Off<T> O;   // the first site; nb[0], nb[1]: the sites right and left of the pair
    bool l, r;  // the left (right) neighbour is not the last (first) site of the lane below (above)
};

template <typename T>
__device__ __forceinline__ PairAt<T> pair_at(const Geom &G, int s)
{
    Nbr S = nbr_of(G, s);
    S.nb[0] = S.x + 2 == G.nx ? s + 2 - G.nx : s + 2;
    PairAt<T> A;
    A.O = offsets<T>(S);
    const int lane = int(threadIdx.x) & 63;
    A.l = lane == 0 || S.x == 0;
    A.r = lane == 63 || S.x + 2 == G.nx;
    return A;
}

template <int CTRL, typename T>
__device__ __forceinline__ T lane_shift(T v)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
    } else {
        Two<int> w = __builtin_bit_cast(Two<int>, v);
        w.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, false);
        w.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, false);
        return __builtin_bit_cast(T, w);
    }
}
template <typename T>
__device__ __forceinline__ T from_below(T v) { return lane_shift<0x138>(v); }  // lane i: lane i - 1's
template <typename T>
__device__ __forceinline__ T from_above(T v) { return lane_shift<0x130>(v); }  // lane i: lane i + 1's

template <typename T>
__device__ __forceinline__ Two<T> two(const T *P, unsigned b)
{
    return *reinterpret_cast<const Two<T> *>(at(P, b));
}

// The rows of NC components at a pair and its neighbours.
template <typename T, int NC>
struct PairRows {
    Two<T> c[NC], yp[NC], ym[NC], zp[NC], zm[NC];
    T l[NC], r[NC];

    __device__ __forceinline__ void load(const T *__restrict__ F, int N, const PairAt<T> &A)
    {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const T *P = plane(F, k, N);
            c[k] = two(P, A.O.s);
            yp[k] = two(P, A.O.nb[2]);
            ym[k] = two(P, A.O.nb[3]);
            zp[k] = two(P, A.O.nb[4]);
            zm[k] = two(P, A.O.nb[5]);
        }
        if (A.l)
#pragma unroll
            for (int k = 0; k < NC; ++k) l[k] = *at(plane(F, k, N), A.O.nb[1]);
        if (A.r)
#pragma unroll
            for (int k = 0; k < NC; ++k) r[k] = *at(plane(F, k, N), A.O.nb[0]);
    }
    __device__ __forceinline__ void edges(const PairAt<T> &A)
    {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const T a = from_below(c[k].y), b = from_above(c[k].x);
            l[k] = A.l ? l[k] : a;
            r[k] = A.r ? r[k] : b;
        }
    }
};

// gather_q and gather_u at site h (0, 1) of the pair.
template <typename T>
__device__ __forceinline__ void pair_q(const PairRows<T, 5> &F, int h, T q[5], T d[3][5], T lap[5])
{
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        q[k] = F.c[k][h];
        stencil7(q[k], h ? F.r[k] : F.c[k].y, h ? F.c[k].x : F.l[k], F.yp[k][h], F.ym[k][h], F.zp[k][h], F.zm[k][h],
                 d[0][k], d[1][k], d[2][k], lap[k]);
    }
}

template <typename T>
__device__ __forceinline__ void pair_u(const PairRows<T, 3> &F, int h, T uc[3], T W[3][3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        uc[a] = F.c[a][h];
        W[a][0] = T(0.5) * ((h ? F.r[a] : F.c[a].y) - (h ? F.c[a].x : F.l[a]));
        W[a][1] = T(0.5) * (F.yp[a][h] - F.ym[a][h]);
        W[a][2] = T(0.5) * (F.zp[a][h] - F.zm[a][h]);
    }
}

// What site_rhs takes at one site of a pair.
template <typename T>
struct SiteIn {
    T q[5], d[3][5], lap[5], uc[3], W[3][3];
};

// A value that the compiler takes as new from here on, after what is held before.
template <typename T>
__device__ __forceinline__ void hold(T &v)
{
    asm volatile("" : "+v"(v));
}

// R at both sites of a pair, one after the other: left to itself the compiler
// runs the two side by side, and their 260 registers leave a SIMD one wave.
template <typename T>
__device__ __forceinline__ void pair_rhs(const Coef<T> &c, SiteIn<T> (&I)[2], T (&R)[2][5])
{
    site_rhs(c, I[0].q, I[0].d, I[0].lap, I[0].uc, I[0].W, R[0]);
#pragma unroll
    for (int k = 0; k < 5; ++k) hold(R[0][k]);
    SiteIn<T> &J = I[1];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        hold(J.q[k]);
        hold(J.lap[k]);
#pragma unroll
        for (int e = 0; e < 3; ++e) hold(J.d[e][k]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        hold(J.uc[a]);
#pragma unroll
        for (int e = 0; e < 3; ++e) hold(J.W[a][e]);
    }
    site_rhs(c, J.q, J.d, J.lap, J.uc, J.W, R[1]);
}

// pred_at and corr_at at both sites of a pair (the pair's first site s; mine:
// write them).
template <typename T>
__device__ __forceinline__ void pair_in(const PairAt<T> &A, int N, const T *__restrict__ Q, const T *__restrict__ u,
                                        SiteIn<T> (&I)[2])
{
    PairRows<T, 5> FQ;
    PairRows<T, 3> FU;
    FQ.load(Q, N, A);
    FU.load(u, N, A);
    FQ.edges(A);
    FU.edges(A);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        pair_q(FQ, h, I[h].q, I[h].d, I[h].lap);
        pair_u(FU, h, I[h].uc, I[h].W);
    }
}

template <typename T>
__device__ __forceinline__ void pred_pair(const Geom &G, const Coef<T> &c, const T *__restrict__ Q,
                                          const T *__restrict__ u, T *__restrict__ Qs, int s, bool mine)
{
    const int N = G.N;
    const PairAt<T> A = pair_at<T>(G, s);
    SiteIn<T> I[2];
    T R[2][5];
    pair_in(A, N, Q, u, I);
    pair_rhs(c, I, R);
    if (mine)
#pragma unroll
        for (int k = 0; k < 5; ++k)
            *reinterpret_cast<Two<T> *>(at(plane(Qs, k, N), A.O.s)) = Two<T>{I[0].q[k] + R[0][k], I[1].q[k] + R[1][k]};
}

template <typename T>
__device__ __forceinline__ void corr_pair(const Geom &G, const Coef<T> &c, T *__restrict__ Q,
                                          const T *__restrict__ Qs, const T *__restrict__ u, int s, bool mine)
{
    const int N = G.N;
    const PairAt<T> A = pair_at<T>(G, s);
    SiteIn<T> I[2];
    T R[2][5];
    Two<T> qn[5];
    pair_in(A, N, Qs, u, I);
    pair_rhs(c, I, R);
#pragma unroll
    for (int k = 0; k < 5; ++k) qn[k] = two(static_cast<const T *>(plane(Q, k, N)), A.O.s);
    if (mine)
#pragma unroll
        for (int k = 0; k < 5; ++k)
            *reinterpret_cast<Two<T> *>(at(plane(Q, k, N), A.O.s)) =
                Two<T>{T(0.5) * (qn[k].x + I[0].q[k] + R[0][k]), T(0.5) * (qn[k].y + I[1].q[k] + R[1][k])};
}

// Free-energy density at one site (Eq. (1) with the divergence term).
template <typename T>
__device__ __forceinline__ T fdens_at(const Geom &G, const Coef<T> &c, const T *__restrict__ Q, int s)
{
    const Off<T> O = offsets<T>(nbr_of(G, s));
    T q[5], d[3][5], lap[5], Qf[3][3], dQ[3][3][3], CQ[3][3], Q2[3][3], M[3][3], div[3];
    gather_q(Q, G.N, O, q, d, lap);
    full3(q, Qf);
    full_grad(d, dQ);
    curl(dQ, CQ);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            Q2[a][b] = Qf[a][0] * Qf[0][b] + Qf[a][1] * Qf[1][b] + Qf[a][2] * Qf[2][b];
            M[a][b] = CQ[a][b] + c.q0x2 * Qf[a][b];
        }
        div[a] = dQ[0][a][0] + dQ[1][a][1] + dQ[2][a][2];
    }
    return free_energy(c, Qf, Q2, Q2[0][0] + Q2[1][1] + Q2[2][2], div, M);
}

template <typename T>
Coef<T> make_coef(const PhysParams &p)
{
    Coef<T> c;
    c.a = T(p.A0 * (1.0 - p.gamma / 3.0));
    c.bg = T(p.A0 * p.gamma);
    c.K = T(p.K);
    c.q0x2 = T(2.0 * p.q0);
    c.Kq0x2 = T(2.0 * p.K * p.q0);
    c.Kq0sq4 = T(4.0 * p.K * p.q0 * p.q0);
    c.xi = T(p.xi);
    c.Gamma = T(p.Gamma);
    c.rho0 = T(p.rho0);
    c.omega = T(1.0 / p.tau);
    c.pref = T(1.0 - 0.5 / p.tau);
    return c;
}

}  // namespace hlb
