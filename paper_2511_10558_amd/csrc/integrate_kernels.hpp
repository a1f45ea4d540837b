// What the persistent kernels share: taking cells from the queue, the launch's
// time, the phase clocks, and the kernel for cells of more than 64 species
// (instantiated per precision form in a source file of its own).
#pragma once

#include "device_step.hpp"

namespace abdf {

// A persistent kernel and its launch shape.
struct Persistent {
    const void *fn;
    int threads;
    size_t lds;            // dynamic
    size_t fixed;          // static
    bool defers = false;   // puts cells on FP64 factors back (kDefer)
    size_t total() const { return lds + fixed; }
};

// Static LDS of a persistent kernel: StepLds and the phase clocks.
template <int W>
constexpr size_t kFixedLds = sizeof(StepLds<W>) + kPhases * sizeof(unsigned long long);
Persistent integrate_wide_fp64(const DeviceNet &n);
Persistent integrate_wide_fp32(const DeviceNet &n);
// for networks of at most 64 species; fp64_too: the FP32-LU form whose LDS also
// holds FP64 factors
Persistent integrate_tiny(const DeviceNet &n, int prec, bool fp64_too);
Persistent reverse_kernel(const DeviceNet &n);

// Eight waves to a workgroup: one thread per species up to 512.
constexpr int kIntegrateWaves = 8;

// Accumulated time of the phases of one workgroup (thread 0's clock).
struct PhaseClock {
    bool on;
    unsigned long long last;
    __device__ __forceinline__ void start() {
        if (on) last = wall_clock64();
    }
    __device__ __forceinline__ void stop(unsigned long long *sum) {
        if (on) {
            const unsigned long long t = wall_clock64();
            *sum += t - last;
            last = t;
        }
    }
};

// Whether this workgroup puts its cell back and ends: the launch's time is up,
// or (when cells wait on the host for slots, or for the form that holds FP64
// factors) another workgroup found the queue empty; a server's launch also ends
// when the host calls.  Uniform; contains a barrier.
template <int W>
__device__ __forceinline__ bool time_up(const Slots &s, const IntegrateArgs &a, unsigned long long t0,
                                        StepLds<W> &L) {
    if (threadIdx.x == 0) {
        const unsigned long long ran = wall_clock64() - t0;
        bool up = ran > a.ticks;
        if ((a.flags & kStopOnIdle) || ((a.flags & kDefer) && (L.cs.n_attempts & 7) == 0))   // not a load of every short attempt
            up |= __hip_atomic_load(&s.q->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.launch;
        // host memory is some 2 us away: not every attempt (of 50 us and more, or 20 us of a wave alone)
        if ((a.flags & kServe) && (L.cs.n_attempts & (W == 1 ? 15 : 3)) == 0 && ran > s.q->ticks_call)
            up |= __hip_atomic_load(s.q->call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0;
        L.flag = up;
    }
    __syncthreads();
    return L.flag != 0;
}

// Takes the next slot into L.slot (-1: none) and its control block into L.cs.
template <int W>
__device__ __forceinline__ int take_slot(const Slots &s, const IntegrateArgs &a, StepLds<W> &L) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const int slot = next_slot(s, a.held_limit);
        L.slot = slot;
        if (slot >= 0)
            L.cs = s.ctl[slot];
        else if ((a.flags & kStopOnIdle) ||
                 ((a.flags & kDefer) && __hip_atomic_load(&s.q->n64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0))
            __hip_atomic_store(&s.q->stop, a.launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(L.slot);   // a scalar: so are the slot's addresses
}

// Integrates queued cells.  One workgroup per compute unit (the factorisation's
// accumulators take its registers); the dynamic LDS serves the factorisation,
// the residual and the solves in turn.
template <int W, bool kF32>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2)))
k_integrate(Slots s, DeviceNet n, IntegrateArgs a) {
    extern __shared__ double smem[];
    __shared__ StepLds<W> L;
    __shared__ unsigned long long t_phase[kPhases];
    const unsigned long long t0 = wall_clock64();
    if (threadIdx.x < kPhases) t_phase[threadIdx.x] = 0;
    const bool rk = s.method == ABDF_METHOD_ESDIRK5;
    PhaseClock clk{(a.flags & kProf) && threadIdx.x == 0, 0};
    while (true) {
        const int slot = take_slot<W>(s, a, L);
        if (slot < 0) break;
        SpeciesState y;
        load_rows(s, slot, y);
        bool up = false;
        while (true) {
            clk.start();
            if (rk)
                begin_stage_rk<W>(s, slot, L, y);
            else
                begin_attempt<W>(s, n, slot, L, y);
            if (L.cs.status != kRunning) break;
            store_rows(s, slot, y);   // the factorisation needs the registers
            clk.stop(&t_phase[kPhaseControl]);
            if (!L.cs.lu_valid) {
                if (kF32 && L.cs.lu_mode != kLu64)
                    factor_slot<float, W>(s, n, slot, L.cs, smem);
                else
                    factor_slot<double, W>(s, n, slot, L.cs, smem);
                if (threadIdx.x == 0) {
                    L.cs.c_lu = L.cs.c;
                    L.cs.lu_valid = 1;
                    L.cs.jv_valid = 1;
                    L.cs.n_lu += 1;
                    if (kF32 && L.cs.lu_mode == kLu64) L.cs.n_lu64 += 1;
                }
                __syncthreads();
                clk.stop(&t_phase[kPhaseFactor]);
            }
            const int phase = newton_slot<W, kF32>(s, n, slot, L, y, smem, clk.on ? &t_phase[kPhaseRhs] : nullptr);
            clk.stop(&t_phase[kPhaseNewton]);
            load_rows(s, slot, y);
            if (rk)
                control_rk<W>(s, L, y, phase, smem);
            else
                control_bdf<W>(s, slot, L, y, phase, smem);
            if (L.cs.status != kRunning) break;
            up = time_up<W>(s, a, t0, L);
            clk.stop(&t_phase[kPhaseControl]);
            if (up) break;
        }
        store_rows(s, slot, y);
        if (!up) finish_slot(s, slot, L.cs, L.cs.status);
        __syncthreads();
        if (threadIdx.x == 0) {
            s.ctl[slot] = L.cs;
            if (up) hold_slot(s, slot);
        }
        if (up) break;
    }
    __syncthreads();
    if ((a.flags & kProf) && threadIdx.x < kPhases)
        atomicAdd(&s.q->ticks[threadIdx.x],
                  t_phase[threadIdx.x] - (threadIdx.x == kPhaseNewton ? t_phase[kPhaseRhs] : 0ull));
}

template <bool kF32>
Persistent integrate_wide(const DeviceNet &n) {
    constexpr int W = kIntegrateWaves;
    const size_t lu = std::max(lu2_lds_bytes<double, W>(n.NP), kF32 ? lu2_lds_bytes<float, W>(n.NP) : size_t(0));
    // corrector: b, z (and z2), x, then the rates or the solve's scratch or
    // the folded norms' 512 values
    const size_t newton = sizeof(double) * ((kF32 ? 3 : 2) * size_t(n.NP) + n.S +
                                            std::max({size_t(n.R), kLuW + size_t(n.NP) / 2, size_t(512)}));
    return {(const void *)&k_integrate<W, kF32>, 64 * W, std::max(lu, newton), kFixedLds<W>};
}

}  // namespace abdf
