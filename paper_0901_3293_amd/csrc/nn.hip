// nn.hip -- kernels of the 3D convolutional surrogate on BF16 matrix cores.
//
// Activations are channels-last bfloat16, act[site][C] with C padded to 16 or
// 32.  tap = kz*9 + ky*3 + kx of a 3x3x3 kernel reads the input at offset
// (kx-1, ky-1, kz-1), periodic.  The convolutions are implicit GEMMs on
// v_mfma_f32_16x16x32_bf16 with FP32 accumulation (k_conv); the weight
// gradient is a GEMM over sites (k_wgrad) with a deterministic FP64 reduction
// of per-block partials.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "nn.h"
#include "tiles.h"

namespace hlb {
namespace nn {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int BLK = 256;

__device__ __forceinline__ unsigned short f2bf(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                                    // round to nearest even
    return (unsigned short)(u >> 16);
}

// Two values rounded to nearest even in one instruction (a in the low half).
__device__ __forceinline__ unsigned f2bf2(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// K = 32 slices of the nine (y, z) taps of one x-offset, times three: the 32
// input channels of one tap, or the 16 channels of two taps.
constexpr int nksteps(int cin) { return cin == 32 ? 27 : 15; }

// Weights of one layer in MFMA fragment order for k_conv, from the flat FP32
// parameters W[co][ci][tap].  A convolution as run maps CIN input channels to
// COUT output channels; its fragment array is [kstep][COUT/16][lane][8] bf16,
// lane = 16 lg + i holding output channel 16 ns + i and the 8 input channels
// that lane group lg contributes to the K = 32 slice of the kstep.  Ksteps run
// x-offset major: for CIN = 32 kstep dx*9 + (dz*3 + dy) is one tap; for
// CIN = 16 kstep dx*5 + p pairs the (dz, dy) positions 2p (lane groups 0-1)
// and 2p + 1 (lane groups 2-3; zero past the ninth).
// Forward (transposed = 0): out channel co, in channel ci, tap as stored.
// Backward-data (transposed = 1): out channel ci, in channel co, tap reversed
// (offset -> -offset), i.e. the adjoint convolution.
// One launch for all of a step's fragment arrays (blockIdx.y): an array takes
// less time than the launch, 4.6 us each for the eight of four layers, 37 us of a
// training step, and together 6.
__global__ __launch_bounds__(BLK) void k_wprep(WeightArrays a)
{
    const float *__restrict__ W = a.of[blockIdx.y].W;
    unsigned short *__restrict__ F = a.of[blockIdx.y].F;
    const int CI = a.of[blockIdx.y].CI, CO = a.of[blockIdx.y].CO;
    const int cin = a.of[blockIdx.y].cin, cout = a.of[blockIdx.y].cout, transposed = a.of[blockIdx.y].transposed;
    const int nks = nksteps(cin), ns_n = cout / 16;
    const int total = nks * ns_n * 64 * 8;
    for (int e = blockIdx.x * BLK + threadIdx.x; e < total; e += gridDim.x * BLK) {
        const int j = e & 7, lane = (e >> 3) & 63, rest = e >> 9;
        const int ns = rest % ns_n, ks = rest / ns_n;
        const int lg = lane >> 4, i = lane & 15;
        int dx, q, c;
        if (cin == 32) {
            dx = ks / 9;
            q = ks % 9;
            c = 8 * lg + j;
        } else {
            dx = ks / 5;
            q = 2 * (ks % 5) + (lg >= 2 ? 1 : 0);
            c = 8 * (lg & 1) + j;
        }
        const int o = 16 * ns + i;
        float v = 0.f;
        if (q < 9) {
            const int tap = (q / 3) * 9 + (q % 3) * 3 + dx;
            if (!transposed) {
                if (o < CO && c < CI) v = W[(o * CI + c) * 27 + tap];
            } else {
                if (o < CI && c < CO) v = W[(c * CI + o) * 27 + (26 - tap)];
            }
        }
        F[e] = f2bf(v);
    }
}

// Network inputs (NIN = 18 channels): Q (5 stored components), u (3), the
// last increment d1 = Q(t) - Q(t-k) (5) and its change s2 = Q(t) - 2 Q(t-k) +
// Q(t-2k) (5).  Standardised with norm and rounded to bf16 into the first
// layer's [N][32] activation (channels 18..31 zero).
__device__ __forceinline__ void store_input_row(int N, int s, const float v[NIN], const float *__restrict__ norm,
                                                unsigned short *__restrict__ A0)
{
    alignas(16) unsigned short h[32];
#pragma unroll
    for (int c = 0; c < 32; ++c) h[c] = c < NIN ? f2bf((v[c] - norm[NORM_IN_MEAN + c]) / norm[NORM_IN_STD + c]) : 0;
    uint4 *dst = reinterpret_cast<uint4 *>(A0 + size_t(s) * 32);
    const uint4 *src = reinterpret_cast<const uint4 *>(h);
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[k] = src[k];
}

// From raw inputs x [NIN][N] FP32.
__global__ __launch_bounds__(BLK) void k_pack(int N, const float *__restrict__ x, const float *__restrict__ norm,
                                              unsigned short *__restrict__ A0)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    if (s >= N) return;
    float v[NIN];
#pragma unroll
    for (int c = 0; c < NIN; ++c) v[c] = x[size_t(c) * N + s];
    store_input_row(N, s, v, norm, A0);
}

// From a solver state (Q, u of type T) and the history (d1, s2 FP32 [5][N]).
template <typename T>
__global__ __launch_bounds__(BLK) void k_pack_state(int N, const T *__restrict__ Q, const T *__restrict__ u,
                                                    const float *__restrict__ d1, const float *__restrict__ s2,
                                                    const float *__restrict__ norm, unsigned short *__restrict__ A0)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    if (s >= N) return;
    float v[NIN];
#pragma unroll
    for (int c = 0; c < 5; ++c) v[c] = float(Q[size_t(c) * N + s]);
#pragma unroll
    for (int c = 0; c < 3; ++c) v[5 + c] = float(u[size_t(c) * N + s]);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        v[8 + c] = d1[size_t(c) * N + s];
        v[13 + c] = s2[size_t(c) * N + s];
    }
    store_input_row(N, s, v, norm, A0);
}

// Raw inputs [NIN][N] from a solver state and the history.
template <typename T>
__global__ __launch_bounds__(BLK) void k_inputs(int N, const T *__restrict__ Q, const T *__restrict__ u,
                                                const float *__restrict__ d1, const float *__restrict__ s2,
                                                float *__restrict__ x)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    if (s >= N) return;
#pragma unroll
    for (int c = 0; c < 5; ++c) x[size_t(c) * N + s] = float(Q[size_t(c) * N + s]);
#pragma unroll
    for (int c = 0; c < 3; ++c) x[size_t(5 + c) * N + s] = float(u[size_t(c) * N + s]);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        x[size_t(8 + c) * N + s] = d1[size_t(c) * N + s];
        x[size_t(13 + c) * N + s] = s2[size_t(c) * N + s];
    }
}

// History from three snapshots of Q (type T) k steps apart, oldest A, then
// B, then the current Q: d1 = Q - B, s2 = Q - 2B + A (in T, then FP32).
template <typename T>
__global__ __launch_bounds__(BLK) void k_hist3(int N, const T *__restrict__ Q, const T *__restrict__ B,
                                               const T *__restrict__ A, float *__restrict__ d1,
                                               float *__restrict__ s2)
{
    const size_t i = size_t(blockIdx.x) * BLK + threadIdx.x;
    if (i >= size_t(5) * N) return;
    const T q = Q[i], b = B[i], a = A[i];
    d1[i] = float(q - b);
    s2[i] = float((q - b) - (b - a));
}

// History after k plain steps from the snapshot P: dq = Q - P, s2 = dq - d1, d1 = dq.
template <typename T>
__global__ __launch_bounds__(BLK) void k_hist_step(int N, const T *__restrict__ Q, const T *__restrict__ P,
                                                   float *__restrict__ d1, float *__restrict__ s2)
{
    const size_t i = size_t(blockIdx.x) * BLK + threadIdx.x;
    if (i >= size_t(5) * N) return;
    const float dq = float(Q[i] - P[i]);
    s2[i] = dq - d1[i];
    d1[i] = dq;
}

// Increment predicted by the network: dq = d1 + beta s2 + (y std + mean), y
// the standardised network output [N][5].
__device__ __forceinline__ float predicted(const float *__restrict__ Y, const float *__restrict__ norm, int N, int s,
                                           int k, float d1, float s2)
{
    return d1 + norm[NORM_BETA] * s2 + (Y[size_t(s) * 5 + k] * norm[NORM_OUT_STD + k] + norm[NORM_OUT_MEAN + k]);
}

// dq [5][N] from raw inputs x (history in its channels 8..17).
__global__ __launch_bounds__(BLK) void k_predict_out(int N, const float *__restrict__ Y, const float *__restrict__ norm,
                                                     const float *__restrict__ x, float *__restrict__ dq)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    if (s >= N) return;
#pragma unroll
    for (int k = 0; k < 5; ++k)
        dq[size_t(k) * N + s] =
            predicted(Y, norm, N, s, k, x[size_t(8 + k) * N + s], x[size_t(13 + k) * N + s]);
}

// One network jump on a solver state: dq from the history; either written
// out (dq != nullptr) or applied: Q += dq, s2 = dq - d1, d1 = dq.
template <typename T>
__global__ __launch_bounds__(BLK) void k_jump(int N, const float *__restrict__ Y, const float *__restrict__ norm,
                                              float *__restrict__ d1, float *__restrict__ s2, T *__restrict__ Q,
                                              float *__restrict__ dq)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    if (s >= N) return;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const size_t i = size_t(k) * N + s;
        const float a = d1[i], b = s2[i];
        const float d = predicted(Y, norm, N, s, k, a, b);
        if (dq) {
            dq[i] = d;
        } else {
            Q[i] = T(Q[i] + T(d));
            s2[i] = d - a;
            d1[i] = d;
        }
    }
}

// Loss and its gradient: target t = (dq - d1 - beta s2 - mean) / std with the
// history from x, d = y - t, dZ = bf16(2 d / (5 N)), block partials of
// sum d^2 (FP64).
__global__ __launch_bounds__(BLK) void k_lossgrad(int N, const float *__restrict__ Y, const float *__restrict__ dq,
                                                  const float *__restrict__ x, const float *__restrict__ norm,
                                                  unsigned short *__restrict__ dZ, double *__restrict__ part)
{
    const int s = blockIdx.x * BLK + threadIdx.x;
    double acc = 0.0;
    if (s < N) {
        const float sc = 2.0f / (5.0f * float(N));
        alignas(16) unsigned short h[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (k < 5) {
                const float c = dq[size_t(k) * N + s] - x[size_t(8 + k) * N + s] -
                                norm[NORM_BETA] * x[size_t(13 + k) * N + s];
                const float t = (c - norm[NORM_OUT_MEAN + k]) / norm[NORM_OUT_STD + k];
                const float d = Y[size_t(s) * 5 + k] - t;
                acc += double(d) * double(d);
                h[k] = f2bf(d * sc);
            } else {
                h[k] = 0;
            }
        }
        uint4 *dst = reinterpret_cast<uint4 *>(dZ + size_t(s) * 16);
        const uint4 *src = reinterpret_cast<const uint4 *>(h);
        dst[0] = src[0];
        dst[1] = src[1];
    }
    __shared__ double buf[BLK];
    buf[threadIdx.x] = acc;
    __syncthreads();
    for (int w = BLK / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) buf[threadIdx.x] += buf[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = buf[0];
}

__global__ __launch_bounds__(BLK) void k_sum(const double *__restrict__ part, int n, double *__restrict__ out)
{
    __shared__ double buf[BLK];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += BLK) s += part[i];
    buf[threadIdx.x] = s;
    __syncthreads();
    for (int w = BLK / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) buf[threadIdx.x] += buf[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = buf[0];
}

// Adam (Kingma & Ba) on the flat FP32 parameters.
__global__ __launch_bounds__(BLK) void k_adam(int n, float *__restrict__ p, const float *__restrict__ g,
                                              float *__restrict__ m, float *__restrict__ v, float lr, float b1, float b2,
                                              float eps, float c1, float c2)
{
    const int i = blockIdx.x * BLK + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Per-channel sums of x and x^2 over nsamples x [nch][N] FP32 (FP64 partials
// per block, grid = nch x B).
__global__ __launch_bounds__(BLK) void k_stats(const float *__restrict__ data, int nch, int N, int nsamples,
                                               double *__restrict__ part)
{
    const int c = blockIdx.y;
    double s1 = 0.0, s2 = 0.0;
    const size_t per = size_t(nsamples) * N;
    for (size_t k = size_t(blockIdx.x) * BLK + threadIdx.x; k < per; k += size_t(gridDim.x) * BLK) {
        const size_t smp = k / N, s = k - smp * N;
        const double v = data[(smp * nch + c) * N + s];
        s1 += v;
        s2 += v * v;
    }
    __shared__ double b1[BLK], b2[BLK];
    b1[threadIdx.x] = s1;
    b2[threadIdx.x] = s2;
    __syncthreads();
    for (int w = BLK / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) {
            b1[threadIdx.x] += b1[threadIdx.x + w];
            b2[threadIdx.x] += b2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * (c * gridDim.x + blockIdx.x)] = b1[0];
        part[2 * (c * gridDim.x + blockIdx.x) + 1] = b2[0];
    }
}

// Per-channel sums of the training target c = dq - d1 - beta s2 over
// nsamples pairs (x [ns][NIN][N], dq [ns][5][N]); FP64 partials, grid 5 x B.
__global__ __launch_bounds__(BLK) void k_stats_target(const float *__restrict__ x, const float *__restrict__ dq,
                                                      int N, int nsamples, float beta, double *__restrict__ part)
{
    const int c = blockIdx.y;
    double s1 = 0.0, s2 = 0.0;
    const size_t per = size_t(nsamples) * N;
    for (size_t k = size_t(blockIdx.x) * BLK + threadIdx.x; k < per; k += size_t(gridDim.x) * BLK) {
        const size_t smp = k / N, s = k - smp * N;
        const float t = dq[(smp * 5 + c) * N + s] - x[(smp * NIN + 8 + c) * N + s] -
                        beta * x[(smp * NIN + 13 + c) * N + s];
        s1 += double(t);
        s2 += double(t) * double(t);
    }
    __shared__ double b1[BLK], b2[BLK];
    b1[threadIdx.x] = s1;
    b2[threadIdx.x] = s2;
    __syncthreads();
    for (int w = BLK / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) {
            b1[threadIdx.x] += b1[threadIdx.x + w];
            b2[threadIdx.x] += b2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * (c * gridDim.x + blockIdx.x)] = b1[0];
        part[2 * (c * gridDim.x + blockIdx.x) + 1] = b2[0];
    }
}

// Residual sums for || (Qa + dq) - Qb ||^2 and || Qb ||^2 (FP64 block partials).
template <typename T>
__global__ __launch_bounds__(BLK) void k_resid(int N, const T *__restrict__ Qa, const float *__restrict__ dq,
                                               const T *__restrict__ Qb, double *__restrict__ part)
{
    double s1 = 0.0, s2 = 0.0;
    for (size_t k = size_t(blockIdx.x) * BLK + threadIdx.x; k < size_t(5) * N; k += size_t(gridDim.x) * BLK) {
        const double b = double(Qb[k]);
        const double d = double(Qa[k]) + double(dq[k]) - b;
        s1 += d * d;
        s2 += b * b;
    }
    __shared__ double b1[BLK], b2[BLK];
    b1[threadIdx.x] = s1;
    b2[threadIdx.x] = s2;
    __syncthreads();
    for (int w = BLK / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) {
            b1[threadIdx.x] += b1[threadIdx.x + w];
            b2[threadIdx.x] += b2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = b1[0];
        part[2 * blockIdx.x + 1] = b2[0];
    }
}

inline int blocks(size_t n) { return int((n + BLK - 1) / BLK); }

}  // namespace

Grid3 make_grid(int nx, int ny, int nz)
{
    Grid3 g;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.N = nx * ny * nz;
    return g;
}

// One block per CU, a multiple of the 8 XCDs; fewer on lattices of fewer tiles.
int wgrad_grid(const Grid3 &g)
{
    const long long ntiles = (long long)((g.nx + 31) / 32) * ((g.ny + 3) / 4) * ((g.nz + 1) / 2);
    return int(ntiles < WGRAD_BLOCKS ? (ntiles + 7) / 8 * 8 : WGRAD_BLOCKS);
}

size_t frag_bytes(int cin, int cout) { return size_t(nksteps(cin)) * (cout / 16) * 64 * 16; }

namespace {

int device_cus()
{
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
    }
    return cus;
}

// Forward-style periodic 3x3x3 convolution of a CIN-channel activation into
// COUT channels, as an implicit GEMM on v_mfma_f32_16x16x32_bf16: M = 16
// output channels, N = 16 sites of one x-row, K = 32 (the CIN = 32 channels of
// one tap, or the 16 channels of two taps when CIN = 16).
//
// One block of 8 waves per CU takes a run of tiles of 16 x 8 x 4 output sites.
// A wave owns one block of 16 output channels and a sub-tile of 16 x RY x RZ
// sites, and holds the weights of its output channels (27 k-steps, 108
// registers for 32 inputs) for all its tiles, so LDS carries the input rows
// only: every row read (16 sites, one x-offset) feeds up to RY' RZ' = 6 of the
// wave's accumulators.  With the weights in LDS, as this kernel had them
// before, a k-step's weight and row reads took as long as its MFMAs.
// The input brick of a tile (tile plus a one-site periodic halo, 69 KB for 32
// channels) is copied from global memory straight into one of two LDS
// buffers while the tile before it is computed, so no registers hold it and a
// tile takes one barrier.
//
// Bound: the matrix cores, 46.7k cycles of MFMAs per SIMD and layer at 96^3
// of about 77k cycles a wave lives (19 of 32 us; in a network application the
// kernel takes 42 us with its launch and the write-back of its output, 1.16
// PFLOP/s, against 62-72 us before; 32 -> 16: 28 against 45 us; 48 and 32 under the
// profiler).  The rest is the start of a block (its
// weights and first brick) and the epilogues, which the two waves of a SIMD
// reach together.  Nontemporal output stores measured 2% slower.
//
// Every output accumulates its taps x-offset major, then (z, y), in one chain
// of MFMAs, whatever the sub-tile.
//
// Epilogues:
//  MODE_RELU:   out_bf16[s][co] = bf16(relu(acc + b[co])), 0 for co >= co_valid
//  MODE_LINEAR: out_f32[s][co]  = acc + b[co] for co < co_valid (row stride co_valid)
//  MODE_MASK:   out_bf16[s][co] = mask[s][co] > 0 ? bf16(acc) : 0   (backward through ReLU)
//  MODE_RAW:    out_f32[s][co]  = acc (row stride COUT)
constexpr int WBLK = 512;

template <int CIN, int COUT>
struct ConvShape {
    static constexpr int NS = COUT / 16, NKS = nksteps(CIN), KPD = NKS / 3;
    static constexpr int NSUB = WBLK / 64 / NS;                   // waves per output-channel block
    static constexpr int TY = 8, TZ = 4;                          // block tile: 16 x TY x TZ
    static constexpr int RZ = 2, WZ = TZ / RZ, WY = NSUB / WZ, RY = TY / WY;
    static constexpr int BX = 18, BY = TY + 2, BZ = TZ + 2;       // brick
    static constexpr int BN = BX * BY * BZ;
    static constexpr int V = CIN / 8;                             // 16-byte chunks per site
    static constexpr int NCH = (BN * V + WBLK - 1) / WBLK;        // chunks staged per thread
    static_assert(WY * RY == TY && WZ * RZ == TZ && WY * WZ == NSUB, "the waves cover the tile");
};

// LDS position (in 16-byte chunks) of chunk v of the brick site at x = bx
// within the site's chunks.  A 16-byte LDS read takes its 64 lanes in four
// groups of 16 over 64 banks (256 bytes a cycle, measured): lanes 0-3, 12-15
// and 20-27 together, then 4-11, 16-19 and 28-31, and so on 32 higher.  With
// lane 16 lg + li reading chunk lg of site li + dx, a group mixes two chunks;
// flipping bit 1 of the chunk on every other four sites gives the 16 lanes of
// a group 16 different bank quads at every dx (with two chunks per site they
// differ as they are).  The row of the site only adds a constant.
template <int V>
__device__ __forceinline__ int chunk_swizzle(int bx, int v)
{
    return V == 4 ? v ^ (bx >> 1 & 2) : v;
}

// Periodic wrap of a coordinate of a tile's halo-1 brick: -1 and n wrap.  Past
// n, where the tile hangs over the lattice, any site does (no output that is
// written reads it).
__device__ __forceinline__ int halo_wrap(int v, int n)
{
    v += v < 0 ? n : 0;
    v -= v >= n ? n : 0;
    return min(v, n - 1);
}

// Copies 16 bytes per lane from global memory to LDS (lane i to l + 16 i),
// without registers in between; complete once vmcnt has counted it.
__device__ __forceinline__ void copy16_to_lds(const char *gp, u32x4 *l)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gp,
                                     (__attribute__((address_space(3))) void *)l, 16, 0, 0);
}

template <int CIN, int COUT, int MODE>
__global__ __launch_bounds__(WBLK) void k_conv(Grid3 g, int ctx, int cty, int ntiles, int per_block,
                                               const unsigned short *__restrict__ X,
                                               const u32x4 *__restrict__ Wfrag, const float *__restrict__ bias,
                                               void *__restrict__ out, const unsigned short *__restrict__ mask,
                                               int co_valid)
{
    using S = ConvShape<CIN, COUT>;
    constexpr int NS = S::NS, KPD = S::KPD, V = S::V, NCH = S::NCH, RY = S::RY, RZ = S::RZ;
    // whole waves of chunks: the last copies write past the brick, into the pad
    __shared__ u32x4 sB[2][NCH * WBLK];

    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
    const int ns = w % NS, sub = w / NS, wy = sub % S::WY, wz = sub / S::WY;
    const bool upper = lg >= 2;  // CIN = 16: the lane groups of a k-step's second tap
    const int b = xcd_logical_block();
    const int t_begin = b * per_block;
    const int t_end = min(ntiles, t_begin + per_block);
    if (t_begin >= t_end) return;

    auto origin = [&](int t, int &x0, int &y0, int &z0) __attribute__((always_inline)) {
        const int rr = t / ctx;
        x0 = (t - rr * ctx) * 16;
        const int r2 = rr / cty;
        y0 = (rr - r2 * cty) * S::TY;
        z0 = r2 * S::TZ;
    };
    // This thread's chunks of a brick, position e = threadIdx.x + k WBLK: the
    // brick coordinates of the site and the chunk's byte offset in it.
    unsigned where[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const int e = min(int(threadIdx.x) + k * WBLK, S::BN * V - 1);
        const int site = e / V, r = site / S::BX, bx = site - r * S::BX, bz = r / S::BY, by = r - bz * S::BY;
        where[k] = unsigned(bx) | unsigned(by) << 8 | unsigned(bz) << 16 | unsigned(chunk_swizzle<V>(bx, e % V)) << 24;
    }
    // chunk k of the brick at (x0, y0, z0) into buffer `buf`
    auto stage = [&](int x0, int y0, int z0, int buf, int k) __attribute__((always_inline)) {
        const int x = halo_wrap(x0 - 1 + int(where[k] & 255u), g.nx),
                  y = halo_wrap(y0 - 1 + int(where[k] >> 8 & 255u), g.ny),
                  z = halo_wrap(z0 - 1 + int(where[k] >> 16 & 255u), g.nz);
        // below 2^32 bytes: hlbnn_workspace_bytes takes fewer than 2^26 sites
        const unsigned at = unsigned(x + g.nx * (y + g.ny * z)) * (CIN * 2) + (where[k] >> 24) * 16;
        copy16_to_lds(reinterpret_cast<const char *>(X) + at, &sB[buf][k * WBLK + w * 64]);
    };
    int xn, yn, zn;  // origin of the tile being staged
    origin(t_begin, xn, yn, zn);
#pragma unroll
    for (int k = 0; k < NCH; ++k) stage(xn, yn, zn, 0, k);

    bf16x8 W[S::NKS];
#pragma unroll
    for (int ks = 0; ks < S::NKS; ++ks) W[ks] = __builtin_bit_cast(bf16x8, Wfrag[(ks * NS + ns) * 64 + l]);
    const int co = ns * 16 + 4 * lg;  // first of this lane's four output channels
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (MODE == MODE_RELU || MODE == MODE_LINEAR)
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[r] = co + r < co_valid ? bias[co + r] : 0.f;

    // this lane's chunk of the first row of its sub-tile, per x-offset
    int off[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int cv = CIN == 32 ? lg : (lg & 1);
        off[dx] = ((wz * RZ * S::BY + wy * RY) * S::BX + li + dx) * V + chunk_swizzle<V>(li + dx, cv);
    }

    auto next_brick = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    next_brick();
    // One tile; with MORE the brick of tile t + 1 is staged along the way (no
    // branch on it in the unrolled code, so its addresses are computed under
    // the MFMAs).
    auto tile = [&](int t, int buf, auto more_) __attribute__((always_inline)) {
        constexpr bool more = decltype(more_)::value;
        const int xo = xn + li, y0 = yn + wy * RY, z0 = zn + wz * RZ;
        if (more) origin(t + 1, xn, yn, zn);

        const int rows = min(RY, g.ny - y0), planes = min(RZ, g.nz - z0);  // of the sub-tile, inside the lattice
        const unsigned s0 = unsigned(min(xo, g.nx - 1) + g.nx * (min(y0, g.ny - 1) + g.ny * min(z0, g.nz - 1)));
        auto site = [&](int zz, int yy) __attribute__((always_inline)) {
            return s0 + unsigned(g.nx * (yy + g.ny * zz));
        };
        uint2 mk[RZ][RY];
        if (MODE == MODE_MASK)
#pragma unroll
            for (int zz = 0; zz < RZ; ++zz)
#pragma unroll
                for (int yy = 0; yy < RY; ++yy)
                    if (yy < rows && zz < planes)
                        mk[zz][yy] = *reinterpret_cast<const uint2 *>(mask + size_t(site(zz, yy)) * COUT + co);

        f32x4 acc[RZ][RY];
#pragma unroll
        for (int zz = 0; zz < RZ; ++zz)
#pragma unroll
            for (int yy = 0; yy < RY; ++yy) acc[zz][yy] = f32x4{0.f, 0.f, 0.f, 0.f};
        const u32x4 *B = sB[buf];
        if constexpr (CIN == 32) {
            // Input rows plane by plane, x-offset major: each row feeds the
            // outputs it is a tap of, while the rows of the next plane are read.
            constexpr int NP = 3 * (RZ + 2);
            bf16x8 f[2][RY + 2];
            auto read = [&](int p) __attribute__((always_inline)) {
#pragma unroll
                for (int yy = 0; yy < RY + 2; ++yy)
                    f[p & 1][yy] = __builtin_bit_cast(
                        bf16x8, B[off[p / (RZ + 2)] + (p % (RZ + 2) * S::BY + yy) * S::BX * V]);
            };
            read(0);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int dx = p / (RZ + 2), zz = p % (RZ + 2);
#pragma unroll
                for (int yy = 0; yy < RY + 2; ++yy) {
#pragma unroll
                    for (int oz = 0; oz < RZ; ++oz)
#pragma unroll
                        for (int oy = 0; oy < RY; ++oy) {
                            const int dz = zz - oz, dy = yy - oy;
                            if (dz >= 0 && dz < 3 && dy >= 0 && dy < 3)
                                acc[oz][oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    W[dx * KPD + dz * 3 + dy], f[p & 1][yy], acc[oz][oy], 0, 0, 0);
                        }
                    if (yy == 0 && p + 1 < NP) {
                        // issued here and not later, with the other rows' MFMAs to arrive under
                        __builtin_amdgcn_sched_barrier(6);
                        read(p + 1);
                        if (more && p < NCH) stage(xn, yn, zn, buf ^ 1, p);
                        __builtin_amdgcn_sched_barrier(6);
                    }
                }
            }
        } else {
            if (more)
#pragma unroll
                for (int k = 0; k < NCH; ++k) stage(xn, yn, zn, buf ^ 1, k);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                u32x4 f[RZ + 2][RY + 2];
#pragma unroll
                for (int zz = 0; zz < RZ + 2; ++zz)
#pragma unroll
                    for (int yy = 0; yy < RY + 2; ++yy) f[zz][yy] = B[off[dx] + (zz * S::BY + yy) * S::BX * V];
#pragma unroll
                for (int k = 0; k < KPD; ++k)
#pragma unroll
                    for (int oz = 0; oz < RZ; ++oz)
#pragma unroll
                        for (int oy = 0; oy < RY; ++oy) {
                            const int qa = 2 * k, qb = 2 * k + 1;  // (z, y) taps of the k-step; none past the ninth
                            const u32x4 lo = f[oz + qa / 3][oy + qa % 3];
                            const u32x4 hi = qb < 9 ? f[oz + (qb < 9 ? qb / 3 : 0)][oy + qb % 3] : u32x4{0u, 0u, 0u, 0u};
                            acc[oz][oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                W[dx * KPD + k], __builtin_bit_cast(bf16x8, upper ? hi : lo), acc[oz][oy], 0, 0, 0);
                        }
            }
        }
        // the next brick is in LDS, and every wave has read this one; ahead of
        // this tile's stores, which the wait would otherwise include
        if (more) next_brick();
        if (xo < g.nx)
#pragma unroll
            for (int zz = 0; zz < RZ; ++zz)
#pragma unroll
                for (int yy = 0; yy < RY; ++yy) {
                    if (yy >= rows || zz >= planes) continue;
                    const size_t s = site(zz, yy);
                    f32x4 v = acc[zz][yy];
                    if (MODE == MODE_RELU) {
                        // output channels past co_valid: zero weights, zero bias, so zero
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r] + bv[r], 0.f);
                        *reinterpret_cast<uint2 *>(static_cast<unsigned short *>(out) + s * COUT + co) =
                            make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
                    } else if (MODE == MODE_LINEAR) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (co + r < co_valid) static_cast<float *>(out)[s * co_valid + co + r] = v[r] + bv[r];
                    } else if (MODE == MODE_MASK) {
                        const short mh[4] = {short(mk[zz][yy].x & 0xffffu), short(mk[zz][yy].x >> 16),
                                             short(mk[zz][yy].y & 0xffffu), short(mk[zz][yy].y >> 16)};
                        // the mask is a ReLU output, never NaN: positive where its bits are, as an integer
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = mh[r] > 0 ? v[r] : 0.f;
                        *reinterpret_cast<uint2 *>(static_cast<unsigned short *>(out) + s * COUT + co) =
                            make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
                    } else {
                        *reinterpret_cast<float4 *>(static_cast<float *>(out) + s * COUT + co) =
                            make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
    };
    int t = t_begin;
    for (; t + 1 < t_end; ++t) tile(t, (t - t_begin) & 1, std::true_type{});
    tile(t, (t - t_begin) & 1, std::false_type{});
}

template <int CIN, int COUT, int MODE>
hipError_t conv_launch(const Grid3 &g, const unsigned short *X, const unsigned short *W, const float *bias,
                       void *out, const unsigned short *mask, int co_valid, hipStream_t st)
{
    using S = ConvShape<CIN, COUT>;
    const int ctx = (g.nx + 15) / 16, cty = (g.ny + S::TY - 1) / S::TY, ctz = (g.nz + S::TZ - 1) / S::TZ;
    const int ntiles = ctx * cty * ctz;
    // one resident block per CU (the LDS bound), a multiple of the 8 XCDs
    int grid = device_cus();
    grid = ntiles < grid ? ntiles : grid;
    grid = (grid + 7) & ~7;
    const int per_block = (ntiles + grid - 1) / grid;
    k_conv<CIN, COUT, MODE><<<grid, WBLK, 0, st>>>(g, ctx, cty, ntiles, per_block, X,
                                                   reinterpret_cast<const u32x4 *>(W), bias, out, mask, co_valid);
    return hipGetLastError();
}

// Weight gradient dW[tap][ci][co] = sum_s dZ[s][co] X[s + off(tap)][ci] and
// bias gradient db[co] = sum_s dZ[s][co] on v_mfma_f32_16x16x32_bf16: M = 16
// output channels, N = 16 input channels, K = 32 sites of one x-row.
//
// One block of 8 waves per CU takes a run of tiles of 32 x 4 x 2 sites, z
// fastest.  The input planes of a tile (34 x 6 sites, periodic wrap) and its dZ
// lie channel-major in LDS (rows padded to 40 sites): the input in a ring of
// three pairs of z-planes, two of them in use, so that a tile brings in two
// planes and not four (1.6 instead of 3.2 times its sites; with all four, 235
// MB per 96^3 layer, it took 64 us); dZ in two buffers.  The next
// tile's are transposed into LDS between the MFMAs of this tile, from
// registers loaded one tile ahead.  A staged unit is 8 channels of two
// x-neighbouring sites, four units of a site pair in neighbouring lanes, so a
// load instruction touches whole cache lines (64 strided pieces of one line
// each before, which alone took longer than the MFMAs).  Channel 8 v + j is
// plane (COP or 32) / 8 j + v, and planes are 8 dwords apart modulo 32: the 4
// chunks of 8 site pairs that 32 lanes write as dwords fall on 32 banks, and
// the 16 lanes of a 16-byte read's group (see chunk_swizzle) on 64.
//
// A wave owns one (output-channel block, input-channel block) pair for all 27
// taps over a part of the tile's output rows (half with 32 output channels, a
// quarter with 16), and holds the dZ operands of those rows in registers.
// Each input row it reads, as two aligned 16-byte reads shared by the three
// x-offsets (odd offsets take a 16-bit funnel shift; of the second read only
// the first dword is used, but a 4-byte read would meet 4-way bank conflicts),
// meets every output row it is a (y, z) tap of: up to 9 MFMAs per row (3
// before).  The parts are summed in LDS at the end, in a fixed order.
// The bias gradient is summed while dZ is staged (each thread keeps the
// running sums of the channels it stages; the block adds the threads' sums
// per channel in order at the end).
// Per-block FP32 partials; the final sum is FP64 in a fixed order
// (k_wgrad_reduce), so the result is deterministic.
//
// Bound: the matrix cores (19 us of MFMAs at 96^3) with the waits on loads
// and barriers around them: 52 us per 32 -> 32 layer (0.94 PFLOP/s) against 120
// us with 16 x 4 x 4 tiles staged between barriers, 32 -> 16 35 against 75 us (56
// and 38 under the profiler).
template <int COP>
struct WgradShape {
    static constexpr int TX = 32, TY = 4, TZ = 2;
    static constexpr int BX = TX + 2, BY = TY + 2, ROWS = BY * TZ;  // input rows of a plane pair
    static constexpr int XR = 40;                                 // padded input row (sites)
    static constexpr int PAIR = ROWS * XR, RING = 3;              // halfwords of a plane pair; pairs in LDS
    static constexpr int CSX = RING * PAIR + 48;                  // channel strides (halfwords)
    static constexpr int CSD = TX * TY * TZ + 16;
    static_assert((CSX / 2) % 32 == 8 && (CSD / 2) % 32 == 8, "bank-spread channel strides");
    // the channel of plane p of an n-channel array
    __device__ static constexpr int channel_of(int p, int n) { return p % (n / 8) * 8 + p / (n / 8); }
    static_assert(CSX % 8 == 0 && CSD % 8 == 0 && XR % 8 == 0, "16-byte aligned operand rows");
    static constexpr int UX = BX / 2 * ROWS * 4, UD = TX / 2 * TY * TZ * (COP / 8);  // staged units
    static constexpr int NUX = (UX + WBLK - 1) / WBLK;            // input units per thread
    static_assert(UD <= WBLK, "one dZ unit per thread");
    static constexpr int NM = COP / 16, NPAIR = 2 * NM, NQ = WBLK / 64 / NPAIR;  // waves: pairs x parts
    static constexpr int RY = TY * TZ / NQ;                       // output rows of a part (one z-plane)
    static constexpr int PS = 27 * 32 * COP + COP;                // floats of a partial
};

template <int COP>
__global__ __launch_bounds__(WBLK) void k_wgrad(Grid3 g, int ctx, int ctz, int ntiles, int per_block,
                                                const unsigned short *__restrict__ X,
                                                const unsigned short *__restrict__ dZ, float *__restrict__ part)
{
    using S = WgradShape<COP>;
    constexpr int RY = S::RY, NUX = S::NUX;
    struct Lds {
        unsigned short x[32 * S::CSX], d[2][COP * S::CSD];
    };
    __shared__ __attribute__((aligned(16))) Lds lds;

    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
    const int pair = w % S::NPAIR, mt = pair >> 1, nt = pair & 1, q = w / S::NPAIR;
    const int oz = q * RY / S::TY, oy = q * RY % S::TY;  // first output row of the part
    const int b = xcd_logical_block();
    const int t_begin = b * per_block, t_end = min(ntiles, t_begin + per_block);
    float *P = part + size_t(b) * S::PS;

    f32x4 acc[27];
#pragma unroll
    for (int j = 0; j < 27; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float dsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // Unit k of this thread: 8 channels (chunk v) of the sites bx, bx + 1 of
    // row r of a plane pair, and the dword of its first channel there.
    unsigned where[NUX];
    int word[NUX];
#pragma unroll
    for (int k = 0; k < NUX; ++k) {
        const int e = min(int(threadIdx.x) + k * WBLK, S::UX - 1), v = e & 3, p = e >> 2;
        const int r = p / (S::BX / 2), px = p - r * (S::BX / 2), bz = r / S::BY, by = r - bz * S::BY;
        where[k] = unsigned(2 * px) | unsigned(by) << 8 | unsigned(bz) << 16 | unsigned(v) << 24;
        word[k] = v * (S::CSX / 2) + r * (S::XR / 2) + px;
    }
    const int de = min(int(threadIdx.x), S::UD - 1), dv = de % (COP / 8), dp = de / (COP / 8);
    const int dtx = 2 * dp % S::TX, dty = 2 * dp / S::TX % S::TY, dtz = 2 * dp / (S::TX * S::TY);

    u32x4 xa[NUX], xb[NUX], da, db;  // in flight: the units of one tile
    // unit k of the planes zp, zp + 1
    auto load_x = [&](int k, int x0, int y0, int zp) __attribute__((always_inline)) {
        const int x = x0 - 1 + int(where[k] & 255u);
        const int y = halo_wrap(y0 - 1 + int(where[k] >> 8 & 255u), g.ny),
                  z = halo_wrap(zp + int(where[k] >> 16 & 255u), g.nz);
        // below 2^32 bytes: hlbnn_workspace_bytes takes fewer than 2^26 sites
        const unsigned row = unsigned(g.nx * (y + g.ny * z)), c = (where[k] >> 24) * 16;
        const char *base = reinterpret_cast<const char *>(X);
        xa[k] = *reinterpret_cast<const u32x4 *>(base + ((row + unsigned(halo_wrap(x, g.nx))) * 64u + c));
        xb[k] = *reinterpret_cast<const u32x4 *>(base + ((row + unsigned(halo_wrap(x + 1, g.nx))) * 64u + c));
    };
    // dZ of the tile at (x0, y0, z0); zero outside the lattice and past the last tile
    auto load_d = [&](int x0, int y0, int z0, bool live) __attribute__((always_inline)) {
        const int x = x0 + dtx, y = y0 + dty, z = z0 + dtz;
        const bool in = live && y < g.ny && z < g.nz;
        const size_t s = size_t(x) + size_t(g.nx) * (size_t(y) + size_t(g.ny) * z);
        const u32x4 zero = {0u, 0u, 0u, 0u};
        da = in && x < g.nx ? *reinterpret_cast<const u32x4 *>(dZ + s * COP + dv * 8) : zero;
        db = in && x + 1 < g.nx ? *reinterpret_cast<const u32x4 *>(dZ + (s + 1) * COP + dv * 8) : zero;
    };
    // two sites' 8 channels -> one dword per channel, `stride` dwords apart
    auto put = [&](unsigned *d, int stride, const u32x4 &a, const u32x4 &c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[2 * j * stride] = __builtin_amdgcn_perm(c[j], a[j], 0x05040100u);
            d[(2 * j + 1) * stride] = __builtin_amdgcn_perm(c[j], a[j], 0x07060302u);
        }
    };
    auto put_x = [&](int k, int slot) __attribute__((always_inline)) {
        if (int(threadIdx.x) + k * WBLK < S::UX)
            put(reinterpret_cast<unsigned *>(lds.x + slot * S::PAIR) + word[k], 4 * (S::CSX / 2), xa[k], xb[k]);
    };
    auto put_d = [&](int slot) __attribute__((always_inline)) {
        if (int(threadIdx.x) < S::UD) {
            put(reinterpret_cast<unsigned *>(lds.d[slot]) + dv * (S::CSD / 2) + dp, COP / 8 * (S::CSD / 2), da, db);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                dsum[2 * j] += __uint_as_float(da[j] << 16) + __uint_as_float(db[j] << 16);
                dsum[2 * j + 1] += __uint_as_float(da[j] & 0xffff0000u) + __uint_as_float(db[j] & 0xffff0000u);
            }
        }
    };

    // The tiles of a run that lie in one (x, y) column, from z0 up.
    for (int t = t_begin, n; t < t_end; t += n) {
        const int col = t / ctz, cy = col / ctx;
        const int x0 = (col - cy * ctx) * S::TX, y0 = cy * S::TY, z0 = (t - col * ctz) * S::TZ;
        n = min(t_end - t, ctz - (t - col * ctz));
        __syncthreads();  // the last column's planes are no longer read
        // plane pair j holds the planes z0 - 1 + 2 j and z0 + 2 j; tile i reads pairs i and i + 1
#pragma unroll
        for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int k = 0; k < NUX; ++k) load_x(k, x0, y0, z0 - 1 + S::TZ * j);
            if (j < 2)
#pragma unroll
                for (int k = 0; k < NUX; ++k) put_x(k, j);
        }
        load_d(x0, y0, z0, true);
        put_d(0);
        load_d(x0, y0, z0 + S::TZ, n > 1);
        int s0 = 0, s1 = 1, s2 = 2;  // ring slots of the pairs i, i + 1 and i + 2
        for (int i = 0; i < n; ++i) {
            __syncthreads();  // this tile's planes are written, and those replaced now no longer read
            const unsigned short *drow = lds.d[i & 1] + (16 * mt + li) * S::CSD + (oz * S::TY + oy) * S::TX + 8 * lg;
            const unsigned short *xrow[3];  // first input row of the part, per z-offset
#pragma unroll
            for (int dz = 0; dz < 3; ++dz)
                xrow[dz] = lds.x + (16 * nt + li) * S::CSX + 8 * lg + (oz + dz < 2 ? s0 : s1) * S::PAIR
                         + (((oz + dz) & 1) * S::BY + oy) * S::XR;
            bf16x8 A[RY];
#pragma unroll
            for (int y = 0; y < RY; ++y) A[y] = *reinterpret_cast<const bf16x8 *>(drow + y * S::TX);
            constexpr int NR = 3 * (RY + 2);  // input rows of the part
            u32x4 lo[2], hi[2];
            auto read = [&](int r) __attribute__((always_inline)) {
                const unsigned short *rp = xrow[r / (RY + 2)] + r % (RY + 2) * S::XR;
                lo[r & 1] = *reinterpret_cast<const u32x4 *>(rp);
                hi[r & 1] = *reinterpret_cast<const u32x4 *>(rp + 8);
            };
            read(0);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int dz = r / (RY + 2), yi = r % (RY + 2);
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("" : "+v"(hi[r & 1]));  // keeps the read at 16 bytes, and its wait here
                const u32x4 a = lo[r & 1];
                const unsigned h = hi[r & 1][0];
                const u32x4 o[3] = {a,
                                    {__builtin_amdgcn_alignbit(a[1], a[0], 16), __builtin_amdgcn_alignbit(a[2], a[1], 16),
                                     __builtin_amdgcn_alignbit(a[3], a[2], 16), __builtin_amdgcn_alignbit(h, a[3], 16)},
                                    {a[1], a[2], a[3], h}};
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) {
                        const int y = yi - dy;
                        if (y >= 0 && y < RY)
                            acc[dz * 9 + dy * 3 + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                A[y < 0 || y >= RY ? 0 : y], __builtin_bit_cast(bf16x8, o[dx]),
                                acc[dz * 9 + dy * 3 + dx], 0, 0, 0);
                    }
                    if (dx == 0 && r + 1 < NR) {
                        // issued here, with the other x-offsets' MFMAs to arrive under
                        __builtin_amdgcn_sched_barrier(6);
                        read(r + 1);
                        __builtin_amdgcn_sched_barrier(6);
                    }
                }
                // a unit of the next tile goes to LDS, and its registers to the tile after
                // that (past the column's last tile whatever is there: no tile reads it,
                // and its dZ is zero)
                const int k = r / 3 - 1;
                if (r % 3 == 0 && k >= 0 && k < NUX) {
                    put_x(k < 0 ? 0 : k, s2);
                    load_x(k < 0 ? 0 : k, x0, y0, min(z0 - 1 + S::TZ * (i + 3), g.nz));
                } else if (r % 3 == 0 && k == NUX) {
                    put_d(~i & 1);
                    load_d(x0, y0, z0 + S::TZ * (i + 2), i + 2 < n);
                }
            }
            static_assert((NR - 1) / 3 > NUX, "every unit is staged within a tile");
            const int o = s0;
            s0 = s1;
            s1 = s2;
            s2 = o;
        }
    }
    {
        // bias: channel co summed over the threads that stage it, in order
        float *sS = reinterpret_cast<float *>(&lds);
        static_assert(size_t(S::UD) * 8 * sizeof(float) <= sizeof(lds), "bias sums fit the buffers");
        __syncthreads();
        if (int(threadIdx.x) < S::UD)
#pragma unroll
            for (int j = 0; j < 8; ++j) sS[dp * COP + 8 * dv + j] = dsum[j];
        __syncthreads();
        if (int(threadIdx.x) < COP) {
            float s = 0.f;
            for (int t = 0; t < S::UD / (COP / 8); ++t) s += sS[t * COP + threadIdx.x];
            P[27 * 32 * COP + threadIdx.x] = s;
        }
    }
    // the parts of a pair, halved until one is left
    f32x4 *sA = reinterpret_cast<f32x4 *>(&lds);
    static_assert(size_t(WBLK / 128) * 27 * 64 * 16 <= sizeof(lds), "half the waves' accumulators fit the buffers");
#pragma unroll
    for (int n = S::NQ / 2; n >= 1; n /= 2) {
        __syncthreads();
        if (q >= n && q < 2 * n)
#pragma unroll
            for (int j = 0; j < 27; ++j) sA[((w - n * S::NPAIR) * 27 + j) * 64 + l] = acc[j];
        __syncthreads();
        if (q < n)
#pragma unroll
            for (int j = 0; j < 27; ++j) acc[j] += sA[(w * 27 + j) * 64 + l];
    }
    // [pair][tap][lane][4]: lane (li, lg) holds the output channels of planes 16 mt + 4 lg + r and the input
    // channel of plane 16 nt + li
    if (q == 0)
#pragma unroll
        for (int j = 0; j < 27; ++j) reinterpret_cast<f32x4 *>(P)[(pair * 27 + j) * 64 + l] = acc[j];
}

// Sum the per-block partials (FP64, fixed order) into the flat gradient of one
// layer: W[co][ci][tap] (ci < CI, co < CO) then b[co].  A block takes 64
// consecutive values of the partial layout; each of its four waves adds every
// fourth partial, in eight interleaved sums with as many loads in flight, and
// the 32 sums are added in order.  (One thread per value over all partials
// took 26 us for 512 partials of 32 -> 32; this takes 6.4 us for 256.)
__global__ __launch_bounds__(BLK) void k_wgrad_reduce(const float *__restrict__ part, int nblk, int COP, int CI, int CO,
                                                      float *__restrict__ grad)
{
    __shared__ double sum[4][64];
    const int PS = 27 * 32 * COP + COP;
    const int i = threadIdx.x & 63, q = threadIdx.x >> 6, idx = blockIdx.x * 64 + i;
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (idx < PS) {
        int b = q;
        for (; b + 28 < nblk; b += 32)
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] += double(part[size_t(b + 4 * k) * PS + idx]);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (b + 4 * k < nblk) a[k] += double(part[size_t(b + 4 * k) * PS + idx]);
    }
    sum[q][i] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    __syncthreads();
    if (q != 0 || idx >= PS) return;
    const float v = float((sum[0][i] + sum[1][i]) + (sum[2][i] + sum[3][i]));
    if (idx < 27 * 32 * COP) {
        const int r = idx & 3, l = idx >> 2 & 63, pt = idx >> 8, tap = pt % 27, pair = pt / 27;
        using S = WgradShape<32>;
        const int co = S::channel_of(16 * (pair >> 1) + 4 * (l >> 4) + r, COP),
                  ci = S::channel_of(16 * (pair & 1) + (l & 15), 32);
        if (co < CO && ci < CI) grad[(co * CI + ci) * 27 + tap] = v;
    } else {
        const int co = idx - 27 * 32 * COP;
        if (co < CO) grad[CO * CI * 27 + co] = v;
    }
}

template <int COP>
hipError_t wgrad_launch(const Grid3 &g, const unsigned short *X, const unsigned short *dZ, float *part, int ci, int co,
                        float *grad, hipStream_t st)
{
    using S = WgradShape<COP>;
    const int ctx = (g.nx + S::TX - 1) / S::TX, cty = (g.ny + S::TY - 1) / S::TY, ctz = (g.nz + S::TZ - 1) / S::TZ;
    const int ntiles = ctx * cty * ctz, grid = wgrad_grid(g), per_block = (ntiles + grid - 1) / grid;
    k_wgrad<COP><<<grid, WBLK, 0, st>>>(g, ctx, ctz, ntiles, per_block, X, dZ, part);
    k_wgrad_reduce<<<(S::PS + 63) / 64, BLK, 0, st>>>(part, grid, COP, ci, co, grad);
    return hipGetLastError();
}

}  // namespace

hipError_t conv(const Grid3 &g, int cin, int cout, int mode, const unsigned short *X, const unsigned short *W,
                const float *bias, void *out, const unsigned short *mask, int co_valid, hipStream_t st)
{
#define HLB_CONV(CI_, CO_, M_) \
    if (cin == CI_ && cout == CO_ && mode == M_) return conv_launch<CI_, CO_, M_>(g, X, W, bias, out, mask, co_valid, st)
    HLB_CONV(16, 32, MODE_RELU);
    HLB_CONV(32, 32, MODE_RELU);
    HLB_CONV(32, 16, MODE_LINEAR);
    HLB_CONV(16, 32, MODE_LINEAR);
    HLB_CONV(32, 32, MODE_LINEAR);
    HLB_CONV(16, 32, MODE_MASK);
    HLB_CONV(32, 32, MODE_MASK);
    HLB_CONV(16, 32, MODE_RAW);
    HLB_CONV(32, 32, MODE_RAW);
    HLB_CONV(32, 16, MODE_RAW);
#undef HLB_CONV
    return hipErrorInvalidValue;
}

hipError_t wgrad(const Grid3 &g, int cip, int cop, const unsigned short *X, const unsigned short *dZ, float *part,
                 int ci, int co, float *grad, hipStream_t st)
{
    if (cip == 32 && cop == 32) return wgrad_launch<32>(g, X, dZ, part, ci, co, grad, st);
    if (cip == 32 && cop == 16) return wgrad_launch<16>(g, X, dZ, part, ci, co, grad, st);
    return hipErrorInvalidValue;
}

hipError_t wprep(const WeightArrays &a, hipStream_t st)
{
    if (a.n < 1 || a.n > WeightArrays::MOST) return hipErrorInvalidValue;
    k_wprep<<<dim3(64, a.n), BLK, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t pack(int N, const float *x, const float *norm, unsigned short *A0, hipStream_t st)
{
    k_pack<<<blocks(N), BLK, 0, st>>>(N, x, norm, A0);
    return hipGetLastError();
}

hipError_t pack_state(bool fp32, int N, const void *Q, const void *u, const float *d1, const float *s2,
                      const float *norm, unsigned short *A0, hipStream_t st)
{
    if (fp32)
        k_pack_state<float><<<blocks(N), BLK, 0, st>>>(N, static_cast<const float *>(Q),
                                                       static_cast<const float *>(u), d1, s2, norm, A0);
    else
        k_pack_state<double><<<blocks(N), BLK, 0, st>>>(N, static_cast<const double *>(Q),
                                                        static_cast<const double *>(u), d1, s2, norm, A0);
    return hipGetLastError();
}

hipError_t inputs(bool fp32, int N, const void *Q, const void *u, const float *d1, const float *s2, float *x,
                  hipStream_t st)
{
    if (fp32)
        k_inputs<float><<<blocks(N), BLK, 0, st>>>(N, static_cast<const float *>(Q), static_cast<const float *>(u),
                                                   d1, s2, x);
    else
        k_inputs<double><<<blocks(N), BLK, 0, st>>>(N, static_cast<const double *>(Q),
                                                    static_cast<const double *>(u), d1, s2, x);
    return hipGetLastError();
}

hipError_t hist3(bool fp32, int N, const void *Q, const void *B, const void *A, float *d1, float *s2, hipStream_t st)
{
    if (fp32)
        k_hist3<float><<<blocks(size_t(5) * N), BLK, 0, st>>>(N, static_cast<const float *>(Q),
                                                              static_cast<const float *>(B),
                                                              static_cast<const float *>(A), d1, s2);
    else
        k_hist3<double><<<blocks(size_t(5) * N), BLK, 0, st>>>(N, static_cast<const double *>(Q),
                                                               static_cast<const double *>(B),
                                                               static_cast<const double *>(A), d1, s2);
    return hipGetLastError();
}

hipError_t hist_step(bool fp32, int N, const void *Q, const void *P, float *d1, float *s2, hipStream_t st)
{
    if (fp32)
        k_hist_step<float><<<blocks(size_t(5) * N), BLK, 0, st>>>(N, static_cast<const float *>(Q),
                                                                  static_cast<const float *>(P), d1, s2);
    else
        k_hist_step<double><<<blocks(size_t(5) * N), BLK, 0, st>>>(N, static_cast<const double *>(Q),
                                                                   static_cast<const double *>(P), d1, s2);
    return hipGetLastError();
}

hipError_t predict_out(int N, const float *Y, const float *norm, const float *x, float *dq, hipStream_t st)
{
    k_predict_out<<<blocks(N), BLK, 0, st>>>(N, Y, norm, x, dq);
    return hipGetLastError();
}

hipError_t jump(bool fp32, int N, const float *Y, const float *norm, float *d1, float *s2, void *Q, float *dq,
                hipStream_t st)
{
    if (fp32)
        k_jump<float><<<blocks(N), BLK, 0, st>>>(N, Y, norm, d1, s2, static_cast<float *>(Q), dq);
    else
        k_jump<double><<<blocks(N), BLK, 0, st>>>(N, Y, norm, d1, s2, static_cast<double *>(Q), dq);
    return hipGetLastError();
}

hipError_t lossgrad(int N, const float *Y, const float *dq, const float *x, const float *norm, unsigned short *dZ,
                    double *part, double *out, hipStream_t st)
{
    k_lossgrad<<<blocks(N), BLK, 0, st>>>(N, Y, dq, x, norm, dZ, part);
    k_sum<<<1, BLK, 0, st>>>(part, blocks(N), out);
    return hipGetLastError();
}

hipError_t adam(int n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2, float eps, int t,
                hipStream_t st)
{
    const float c1 = 1.f - powf(b1, float(t)), c2 = 1.f - powf(b2, float(t));
    k_adam<<<blocks(n), BLK, 0, st>>>(n, p, g, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t stats(const float *data, int nch, int N, int nsamples, double *part, int nblk, hipStream_t st)
{
    k_stats<<<dim3(nblk, nch), BLK, 0, st>>>(data, nch, N, nsamples, part);
    return hipGetLastError();
}

hipError_t stats_target(const float *x, const float *dq, int N, int nsamples, float beta, double *part, int nblk,
                        hipStream_t st)
{
    k_stats_target<<<dim3(nblk, 5), BLK, 0, st>>>(x, dq, N, nsamples, beta, part);
    return hipGetLastError();
}

hipError_t resid(bool fp32, int N, const void *Qa, const float *dq, const void *Qb, double *part, int nblk,
                 hipStream_t st)
{
    if (fp32)
        k_resid<float><<<nblk, BLK, 0, st>>>(N, static_cast<const float *>(Qa), dq, static_cast<const float *>(Qb),
                                             part);
    else
        k_resid<double><<<nblk, BLK, 0, st>>>(N, static_cast<const double *>(Qa), dq,
                                              static_cast<const double *>(Qb), part);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace hlb
