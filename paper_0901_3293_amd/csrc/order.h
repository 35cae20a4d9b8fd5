// order.h -- largest eigenvalue and its eigenvector of a symmetric traceless
// 3x3 tensor in FP64 (the local order and the director of Sec. 2.1, 2.3), and
// the comparison of that eigenvalue with a threshold.  Host and device, so the
// CPU tests can hold every path to a reference.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>

namespace hlb {

// FP32-accurate reciprocal (the callers' corrections need no more).
__host__ __device__ __forceinline__ double rcp_fast(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return double(__builtin_amdgcn_rcpf(float(x)));
#else
    return double(1.0f / float(x));
#endif
}

__host__ __device__ __forceinline__ double rsqrt64(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return rsqrt(x);
#else
    return 1.0 / sqrt(x);
#endif
}

// Sign of the director: its last non-zero component is positive.
__host__ __device__ __forceinline__ void sign_director(double v0, double v1, double v2, double d[3])
{
    const double sgn = (v2 != 0.0 ? v2 : (v1 != 0.0 ? v1 : v0)) < 0.0 ? -1.0 : 1.0;
    d[0] = sgn * v0;
    d[1] = sgn * v1;
    d[2] = sgn * v2;
}

// The cyclic Jacobi method: plane rotations over the pairs (0,1), (0,2),
// (1,2), each zeroing its off-diagonal entry (tangent of the smaller rotation
// angle), repeated until the off-diagonal mass is below 1e-30 of the squared
// norm nrm (at most 8 sweeps; 4 suffice in practice).  Keeps every eigenvalue
// within a few ulps of |Q| whatever their spacing; the director is the
// rotation's column of the largest diagonal entry.
__host__ __device__ __forceinline__ void order_jacobi(const double q[5], double nrm, double &lam, double d[3])
{
    double A[3][3] = {{q[0], q[1], q[2]}, {q[1], q[3], q[4]}, {q[2], q[4], -q[0] - q[3]}};
    double V[3][3] = {{1.0, 0.0, 0.0}, {0.0, 1.0, 0.0}, {0.0, 0.0, 1.0}};
    const int P[3] = {0, 0, 1}, R[3] = {1, 2, 2};
#pragma unroll 1
    for (int sweep = 0; sweep < 8; ++sweep) {
        const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
        if (!(off > 1e-30 * nrm)) break;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int p = P[k], r = R[k];
            const double apr = A[p][r];
            if (apr == 0.0) continue;
            const double th = (A[r][r] - A[p][p]) / (2.0 * apr);
            const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
            const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const double amp = A[m][p], amr = A[m][r];
                A[m][p] = c * amp - sn * amr;
                A[m][r] = sn * amp + c * amr;
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const double apm = A[p][m], arm = A[r][m];
                A[p][m] = c * apm - sn * arm;
                A[r][m] = sn * apm + c * arm;
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const double vmp = V[m][p], vmr = V[m][r];
                V[m][p] = c * vmp - sn * vmr;
                V[m][r] = sn * vmp + c * vmr;
            }
        }
    }
    // column of the largest diagonal entry, by selects (an index would put V in LDS)
    const bool k1 = A[1][1] > A[0][0], k2 = A[2][2] > (k1 ? A[1][1] : A[0][0]);
    lam = k2 ? A[2][2] : (k1 ? A[1][1] : A[0][0]);
    sign_director(k2 ? V[0][2] : (k1 ? V[0][1] : V[0][0]), k2 ? V[1][2] : (k1 ? V[1][1] : V[1][0]),
                  k2 ? V[2][2] : (k1 ? V[2][1] : V[2][0]), d);
}

// The same where the largest eigenvalue stands clear of the middle one; false
// (nothing written) where it does not, or where |Q| leaves the range of the
// FP32 start.  nrm = tr Q^2 = 6 p^2.
//
// The eigenvalues are 2 p cos((acos r + 2 pi k) / 3), r = det Q / (2 p^3); the
// gap of the two largest is 2 sqrt(3) p sin(x) with r = -cos 3x, so r > -0.99996
// keeps it above 0.01 p.  From this root in FP32 (off by 1e-6 p, and by 2e-5 p at
// that limit) two Newton steps on the characteristic cubic reach FP64 rounding,
// even with reciprocals of FP32 accuracy.  With l so close to the eigenvalue
// the columns of adj(Q - l) are the eigenvector times one of its components
// (error: that of l over the gap); the column of the largest is taken, and the
// Rayleigh quotient of it, written as a correction to l, gives the eigenvalue to
// a few ulps of |Q|.  The cubic gives l to its own rounding over the gap, so the
// column's error grows with the inverse square of the gap; below a gap of 0.5 p
// (r < -0.9) it is taken again from the corrected l, whose error does not grow:
// 3e-15 rms at the limit (2e-13 from the first l, 7e-15 by the Jacobi sweeps).
// About 170 instructions where those take 1000 to 1500, which is what bounds the
// order analysis and the optics.
__host__ __device__ __forceinline__ bool order_separated(const double q[5], double nrm, double &lam, double d[3])
{
    const float pf = sqrtf(float(nrm) * (1.0f / 6.0f));
    if (!(nrm > 1e-24 && nrm < 1e24)) return false;
    // an exact power of two brings p to [1, 2)
    const int ex = ilogbf(pf);
    const double a = ldexp(q[0], -ex), b = ldexp(q[1], -ex), c = ldexp(q[2], -ex), e = ldexp(q[3], -ex),
                 f = ldexp(q[4], -ex), g = -a - e;
    const double J2 = a * a + b * b + c * c + e * e + f * f + a * e;  // tr A^2 / 2
    const double J3 = a * (e * g - f * f) - b * (b * g - f * c) + c * (b * f - e * c);
    const float p = sqrtf(float(J2) * (1.0f / 3.0f));
    const float r = float(J3) * float(rcp_fast(2.0f * p * p * p));
    if (!(r > -0.99996f)) return false;
    double l = double(2.0f * p * cosf(acosf(fminf(r, 1.0f)) * (1.0f / 3.0f)));
#pragma unroll
    for (int n = 0; n < 2; ++n) l -= ((l * l - J2) * l - J3) * rcp_fast(3.0 * l * l - J2);
    double v0, v1, v2, n2, al, el, gl;
    auto column = [&]() __attribute__((always_inline)) {
        al = a - l, el = e - l, gl = g - l;
        const double m00 = el * gl - f * f, m11 = al * gl - c * c, m22 = al * el - b * b;
        const double m01 = c * f - b * gl, m02 = b * f - c * el, m12 = b * c - f * al;
        const bool k0 = m00 >= m11 && m00 >= m22, k1 = m11 >= m22;
        v0 = k0 ? m00 : (k1 ? m01 : m02), v1 = k0 ? m01 : (k1 ? m11 : m12), v2 = k0 ? m02 : (k1 ? m12 : m22);
        n2 = v0 * v0 + v1 * v1 + v2 * v2;
    };
    column();
    const double res = v0 * (al * v0 + b * v1 + c * v2) + v1 * (b * v0 + el * v1 + f * v2) + v2 * (c * v0 + f * v1 + gl * v2);
    l += res * rcp_fast(n2);
    lam = ldexp(l, ex);
    if (r < -0.9f) column();
    const double s = rsqrt64(n2);
    sign_director(v0 * s, v1 * s, v2 * s, d);
    return true;
}

// Largest eigenvalue and director.  Q = 0 gives 0 and (0, 0, 1).
__host__ __device__ __forceinline__ void order_site(const double q[5], double &lam, double d[3])
{
    const double zz = -q[0] - q[3];
    const double nrm = q[0] * q[0] + q[3] * q[3] + zz * zz + 2.0 * (q[1] * q[1] + q[2] * q[2] + q[4] * q[4]);
    if (!(nrm > 0.0)) {
        lam = 0.0;
        d[0] = 0.0;
        d[1] = 0.0;
        d[2] = 1.0;
        return;
    }
    if (!order_separated(q, nrm, lam, d)) order_jacobi(q, nrm, lam, d);
}

// Whether the largest eigenvalue lies below the threshold: it does where
// threshold - Q is positive definite, i.e. its leading minors are positive.  A
// minor within 1e-12 of zero (on the scale of |threshold| + |Q|, a hundred times
// its rounding and that of the eigenvalue) leaves it to order_site, so the two
// always agree; so do scales whose cubes underflow or overflow, NaN and
// infinities (the last two fail every comparison).
__host__ __device__ __forceinline__ bool order_below(const double q[5], double threshold)
{
    const double zz = -q[0] - q[3];
    const double nrm = q[0] * q[0] + q[3] * q[3] + zz * zz + 2.0 * (q[1] * q[1] + q[2] * q[2] + q[4] * q[4]);
    const double a = threshold - q[0], e = threshold - q[3], g = threshold - zz;
    const double b = q[1], c = q[2], f = q[4];
    const double m2 = a * e - b * b;
    const double m3 = g * m2 - (a * f * f + e * c * c + 2.0 * b * c * f);
    const double S = fabs(threshold) + sqrt(nrm), t1 = 1e-12 * S, t2 = t1 * S, t3 = t2 * S;
    if (S > 1e-90 && S < 1e90) {
        if (a > t1 && m2 > t2 && m3 > t3) return true;
        if (a < -t1 || m2 < -t2 || m3 < -t3) return false;
    }
    double lam, d[3];
    order_site(q, lam, d);
    return lam < threshold;
}

}  // namespace hlb
