// Persistent integration kernels: one workgroup takes a cell from the queue and
// carries it, attempt after attempt, until it ends (or the launch's time is
// up), then takes the next.
//
// Every workgroup has its own cell, so nothing waits for another cell: a cell
// that factors its Newton matrix does so while its neighbours iterate, and no
// launch, list or host poll separates the phases of an attempt.  (With one
// launch per phase over all cells, every attempt of 250 cells of 200 species
// took 0.49 ms, the latency of one factorisation, four residuals, four solves
// and a control kernel, although a cell factors in only one attempt of six:
// 224 ms a solve against 63 ms; 512 cells of 500 species 1473 against 795 ms,
// 96 in the FP32-LU form 840 against 230 ms.)
#include "integrate_kernels.hpp"

namespace abdf {

// ------------------------------------------------------------- launchers --

Persistent integrate_wide_fp64(const DeviceNet &n) { return integrate_wide<false>(n); }

// The tiny-cell kernel serves networks of at most 64 species whose tables fit
// in the LDS beside the matrices (in the FP32-LU form, beside FP64 ones: its
// cells may come to need them).
static Persistent integrate_kernel(const DeviceNet &n, int prec, bool fp64_too) {
    if (n.S <= 64 && integrate_tiny(n, prec, true).total() <= kMaxLds) return integrate_tiny(n, prec, fp64_too);
    return prec == ABDF_PREC_FP32_LU ? integrate_wide_fp32(n) : integrate_wide_fp64(n);
}

size_t integrate_lds(const DeviceNet &n, int prec, bool fp64_too) { return integrate_kernel(n, prec, fp64_too).total(); }
size_t reverse_lds(const DeviceNet &n) { return reverse_kernel(n).total(); }

static int resident_per_cu(const Persistent &p) {
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, p.fn, p.threads, p.lds);
    return e == hipSuccess ? nb : 1;   // 0: a workgroup does not fit a compute unit
}

int integrate_resident_per_cu(const DeviceNet &n, int prec, bool fp64_too) {
    return resident_per_cu(integrate_kernel(n, prec, fp64_too));
}
int reverse_resident_per_cu(const DeviceNet &n) { return resident_per_cu(reverse_kernel(n)); }

static hipError_t launch_persistent(const Persistent &p, const Slots &s, const DeviceNet &n, const IntegrateArgs &a,
                                    int grid, hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    if (p.total() > kMaxLds) return hipErrorInvalidValue;
    Slots ss = s;
    DeviceNet nn = n;
    IntegrateArgs aa = a;
    if (p.defers) aa.flags |= kDefer;
    void *args[] = {&ss, &nn, &aa};
    return hipLaunchKernel(p.fn, dim3(unsigned(grid)), dim3(p.threads), args, p.lds, st);
}

hipError_t launch_integrate(const Slots &s, const DeviceNet &n, const IntegrateArgs &a, bool fp64_too, int grid,
                            hipStream_t st) {
    return launch_persistent(integrate_kernel(n, s.prec, fp64_too), s, n, a, grid, st);
}

hipError_t launch_reverse(const Slots &s, const DeviceNet &n, const IntegrateArgs &a, int grid, hipStream_t st) {
    return launch_persistent(reverse_kernel(n), s, n, a, grid, st);
}

}  // namespace abdf
