// Kernel launchers shared by the host engine and the C-ABI layer.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device_common.hpp"
#include "network.hpp"

struct abdf_cell_stats;

namespace abdf {

struct AdmitArgs {
    int count;
    const int32_t *slots;       // [count] target slots
    const long long *cells;     // [count] source cell indices
    const double *T, *nH, *Av, *zeta, *G0, *x0, *t_end;
    const double *rtol_c, *atol_c;  // per-cell tolerances [cells], or null for rtol / atol
    double rtol, atol;
    double newton_tol;          // > 0: used as is; 0: from each cell's rtol
    const double *tc;           // [cells] expansion times of the conditions, or null (constant)
};

struct HarvestArgs {
    int count;
    const int32_t *slots;       // [count] finished slots
    double *x_out;
    int32_t *status;
    abdf_cell_stats *stats;
    int compact;                // 1: results of the i-th finished slot go to index i, else to its cell
};

// Reverse-sweep admission: cells into slots with their loss gradients.
struct AdjArgs {
    int count;
    const int32_t *slots;
    const long long *cells;
    const double *phi;          // [cells][5] T, n_H, A_V, zeta, G0
    const double *dLdx;         // [cells][S] gradient of the loss with respect to x(t_end)
    const int32_t *status;      // [cells] forward outcome; only ABDF_CELL_OK cells are differentiated
};

struct AdjHarvestArgs {
    int count;
    const int32_t *slots;
    double *g_cell;             // [cells][R] dL/dlog alpha, or null
    double *dx0;                // [cells][S] or null
    double *dphi;               // [cells][5] dL/d(T, n_H, A_V, zeta, G0), or null
};

struct PhysArgs {
    const double *T, *nH, *Av, *zeta, *G0;
};

// One launch of the persistent integration (or reverse sweep).  (Short: with 32
// bytes more of arguments, in scalar registers for the whole kernel, the FP32-LU
// solves took 9% longer.)
struct IntegrateArgs {
    unsigned long long held_limit;   // slots put back by earlier launches: Slots::q->held_tail as last read
    unsigned long long ticks;        // workgroups put their cell back once this many 100 MHz ticks have passed
    int32_t launch;                  // number of this launch (> 0)
    int32_t flags;
};
enum {
    kStopOnIdle = 1,   // cells wait on the host: end as soon as a workgroup finds the queue empty
    kProf = 2,         // accumulate SlotQueue::ticks
    kServe = 4,        // a server's: end for SlotQueue::call too
    kDefer = 8         // (set by the launcher) the one-wave FP32-LU form that puts cells on FP64 factors back
};

// LDS bytes per kernel for a network (the persistent kernels': with their static LDS)
inline size_t admit_lds(const DeviceNet &n) { return sizeof(double) * (4 * size_t(n.S) + n.R); }
constexpr size_t kAdmitFixedLds = sizeof(SlotCtl) + (kWaves + 5) * sizeof(double);   // its static LDS
size_t integrate_lds(const DeviceNet &n, int prec, bool fp64_too);
size_t reverse_lds(const DeviceNet &n);

hipError_t launch_admit(const Slots &s, const DeviceNet &n, const AdmitArgs &a, size_t lds, hipStream_t st);
// Integrates (sweeps) the queued slots with grid workgroups.
// fp64_too: the one-wave FP32-LU kernel in the form that also holds FP64 factors.
hipError_t launch_integrate(const Slots &s, const DeviceNet &n, const IntegrateArgs &a, bool fp64_too, int grid,
                            hipStream_t st);
hipError_t launch_reverse(const Slots &s, const DeviceNet &n, const IntegrateArgs &a, int grid, hipStream_t st);
// Their workgroups resident per CU (0: none fits).
int integrate_resident_per_cu(const DeviceNet &n, int prec, bool fp64_too);
int reverse_resident_per_cu(const DeviceNet &n);
hipError_t launch_harvest(const Slots &s, const HarvestArgs &h, hipStream_t st);

hipError_t launch_adj_admit(const Slots &s, const DeviceNet &n, const AdjArgs &a, size_t lds, hipStream_t st);
hipError_t launch_adj_harvest(const Slots &s, const DeviceNet &n, const AdjHarvestArgs &h, hipStream_t st);
hipError_t launch_grad_sum(const double *g_cell, long long cells, int R, double *out, hipStream_t st);
// dL/dphi [cells][5] (T, n_H, A_V, zeta, G0) from per-cell dL/dlog alpha [cells][R].
hipError_t launch_phys_grad(const DeviceNet &n, const PhysArgs &p, long long cells, const double *g_cell,
                            double *out, hipStream_t st);
inline size_t adj_lds(const DeviceNet &n) { return sizeof(double) * (2 * size_t(n.S) + n.R); }

hipError_t launch_rates(const DeviceNet &n, const PhysArgs &p, long long cells, double *k, hipStream_t st);
// The standalone right-hand side: the kernel and grid for a batch (host
// queries only), then its launch.
struct RhsPlan {
    const void *fn = nullptr;
    long long grid = 0;
    int threads = 0;
    size_t lds = 0;
};
hipError_t plan_rhs(const DeviceNet &n, long long cells, RhsPlan &p);
// start, stop: events (or null) the dispatch itself records at the kernel's
// start and end.
hipError_t launch_rhs_planned(const RhsPlan &p, const DeviceNet &n, long long cells, const double *k, const double *x,
                              double *f, hipStream_t st, hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
hipError_t launch_newton_matrix(const DeviceNet &n, long long cells, const double *k, const double *x,
                                const double *c, double *M, hipStream_t st);
// Factorisation in place of a batch of n x n matrices; scratch: bytes.
struct LuFactorPlan {
    const void *fn = nullptr;
    int grid = 0;
    size_t lds = 0, scratch = 0;
};
LuFactorPlan plan_lu_factor(int n, long long batch, int prec);
hipError_t launch_lu_factor(const LuFactorPlan &p, int n, long long batch, double *A, int32_t *perm, int32_t *info,
                            void *scratch, hipStream_t st);
hipError_t launch_lu_solve(int n, long long batch, const double *LU, const int32_t *perm, double *b, hipStream_t st);
size_t dinv_bytes(int NP, int prec);
int lu_leading_dim(int NP);
hipError_t launch_selftest(int *bad, hipStream_t st);
hipError_t launch_fill_i32(int32_t *v, int32_t value, int n, hipStream_t st);

// Largest LDS of one workgroup, static and dynamic together.  The runtime launches
// a kernel that passes it all the same, and the kernel faults: whatever depends on
// the network is checked against it on the host.
constexpr size_t kMaxLds = 160 * 1024;

}  // namespace abdf
