// Host build of hlb_api.cpp for tests/test_api_nomem.py: the read-outs of f(z) and
// of the counts, whose chunk sums come through host memory, when there is none.
// The kernels' launchers are stand-ins that fail (no device is needed), so a call
// that gets its memory ends with HLB_ERR_HIP.  Prints the status of hlb_get_fz and
// hlb_get_order with memory, then without; "threw" for an exception.
#include <cstdio>
#include <cstdlib>
#include <new>

static bool no_memory = false;
void *operator new(std::size_t n)
{
    void *p = no_memory ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new[](std::size_t n) { return operator new(n); }
void *operator new(std::size_t n, const std::nothrow_t &) noexcept { return no_memory ? nullptr : std::malloc(n); }
void *operator new[](std::size_t n, const std::nothrow_t &) noexcept { return no_memory ? nullptr : std::malloc(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
void operator delete[](void *p, std::size_t) noexcept { std::free(p); }

#include "../../paper_0901_3293_amd/csrc/hlb_api.cpp"

namespace hlb {
size_t partial_doubles(int, int, int) { return 1024; }
hipError_t run_init(Device &, const PhysParams &, const double *) { return hipErrorNotSupported; }
hipError_t run_steps(Device &, const PhysParams &, int, KernelTimer *) { return hipErrorNotSupported; }
hipError_t run_readout(Device &, const PhysParams &, double *, double *, double *) { return hipErrorNotSupported; }
size_t readout_partials(const Geom &) { return 0; }
const char *kernel_name(int) { return nullptr; }
int tile_tz_fill(const Device &, int, bool, int) { return 0; }
int fz_parts(const Geom &) { return 2; }
int count_parts(const Geom &) { return 2; }
hipError_t run_fz(Device &, const PhysParams &, double *) { return hipErrorNotSupported; }
hipError_t run_count(Device &, double, int *) { return hipErrorNotSupported; }
hipError_t run_order(Device &, double, double *, double *, unsigned char *, double *) { return hipErrorNotSupported; }
hipError_t run_optics(Device &, const OpticsParams &, double *) { return hipErrorNotSupported; }
}  // namespace hlb

int main()
{
    alignas(256) static char ws[1 << 20];
    double fz[4];
    long long n;
    for (int i = 0; i < 4; ++i) {
        hlb_ctx *c = nullptr;
        if (hlb_create(4, 4, 4, HLB_FP64, ws, sizeof(ws), nullptr, &c) != HLB_OK) return 1;
        c->have_params = c->have_fields = true;
        no_memory = i >= 2;
        int status = 0;
        bool threw = false;
        try {
            status = i % 2 ? hlb_get_order(c, 0.19, nullptr, nullptr, nullptr, nullptr, &n) : hlb_get_fz(c, fz);
        } catch (const std::bad_alloc &) {
            threw = true;
        }
        no_memory = false;
        if (threw)
            std::puts("threw");
        else
            std::printf("%d\n", status);
        hlb_destroy(c);
    }
    return 0;
}
