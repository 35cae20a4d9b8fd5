// Host build of order.h (largest eigenvalue, director and threshold test of a
// symmetric traceless 3x3 tensor) for the CPU test.  Reads n, a threshold and n
// tensors (xx, xy, xz, yy, yz) as doubles; writes per tensor, as doubles:
// eigenvalue and director of order_site, of order_jacobi, whether
// order_separated took the tensor, and order_below.
#include <cstdio>
#include <vector>

#include "../../paper_0901_3293_amd/csrc/order.h"

int main(int argc, char **argv)
{
    if (argc != 3) return 1;
    FILE *f = std::fopen(argv[1], "rb");
    double head[2];
    if (!f || std::fread(head, sizeof(double), 2, f) != 2) return 2;
    const size_t n = size_t(head[0]);
    std::vector<double> q(5 * n), out(10 * n);
    if (std::fread(q.data(), sizeof(double), 5 * n, f) != 5 * n) return 3;
    std::fclose(f);
    for (size_t i = 0; i < n; ++i) {
        const double *t = &q[5 * i];
        double *o = &out[10 * i];
        const double zz = -t[0] - t[3];
        const double nrm = t[0] * t[0] + t[3] * t[3] + zz * zz + 2.0 * (t[1] * t[1] + t[2] * t[2] + t[4] * t[4]);
        double lam, d[3];
        hlb::order_site(t, o[0], o + 1);
        if (nrm > 0.0)
            hlb::order_jacobi(t, nrm, o[4], o + 5);
        else
            o[4] = 0.0, o[5] = 0.0, o[6] = 0.0, o[7] = 1.0;
        o[8] = hlb::order_separated(t, nrm, lam, d);
        o[9] = hlb::order_below(t, head[1]);
    }
    f = std::fopen(argv[2], "wb");
    if (!f || std::fwrite(out.data(), sizeof(double), out.size(), f) != out.size()) return 4;
    return std::fclose(f);
}
