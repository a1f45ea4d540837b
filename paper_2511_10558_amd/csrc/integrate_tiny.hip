// The persistent integration of cells of at most 64 species.
#include "device_tiny.hpp"
#include "integrate_kernels.hpp"

namespace abdf {

// Integrates queued cells of at most 16 kTiles species, one wave per cell
// (TinyCell).
//
// The FP32-LU form (T = float) comes twice.  A cell that falls back to FP64
// factors needs twice the LDS for them, which would halve the cells resident on
// a compute unit between 33 and 48 species (16000 cells of 33 species: 401 ms a
// solve in FP32, 796 in FP64) for the few that do.  So the form without them puts such a
// cell back, counts it in SlotQueue::n64 and ends when it has no other cells;
// the host launches the form with both while there are some.
template <typename T, int kTiles, bool kFp64Too>
__global__ void __launch_bounds__(64) k_integrate_tiny(Slots s, DeviceNet n, IntegrateArgs a) {
    extern __shared__ double smem[];
    __shared__ StepLds<1> L;
    __shared__ unsigned long long t_phase[kPhases];
    const unsigned long long t0 = wall_clock64();
    if (threadIdx.x < kPhases) t_phase[threadIdx.x] = 0;
    const bool rk = s.method == ABDF_METHOD_ESDIRK5;
    PhaseClock clk{(a.flags & kProf) && threadIdx.x == 0, 0};
    constexpr bool kF32 = sizeof(T) == sizeof(float), kPutBack = kF32 && !kFp64Too;
    TinyCell<T, kTiles, kFp64Too> cell(n, reinterpret_cast<unsigned char *>(smem));
    while (true) {
        const int slot = take_slot<1>(s, a, L);
        if (slot < 0) break;
        if (kPutBack && L.cs.lu_mode == kLu64) {
            if (threadIdx.x == 0) hold_slot(s, slot);
            continue;
        }
        const double *kg = s.k + size_t(slot) * n.R;
        SpeciesState y;
        load_rows(s, slot, y);
        cell.load_rates(kg);
        if (L.cs.jv_valid) cell.scatter(n, s.jval + size_t(slot) * n.nnzJ);
        if (L.cs.lu_valid) {
            if (kFp64Too && L.cs.lu_mode == kLu64)
                cell.template restore<double>(s, slot);
            else
                cell.template restore<T>(s, slot);
        }
        bool up = false, put_back = false;
        while (true) {
            clk.start();
            if (rk)
                begin_stage_rk<1>(s, slot, L, y);
            else
                begin_attempt<1>(s, n, slot, L, y);
            if (L.cs.status != kRunning) break;
            if (s.tvar && L.cs.tc > 0.0) cell.load_rates(kg);
            clk.stop(&t_phase[kPhaseControl]);
            if (!L.cs.lu_valid) {
                if (!L.cs.jv_valid)
                    cell.jacobian(n, s.xJ + size_t(slot) * s.S, s.jval + size_t(slot) * n.nnzJ);
                const bool fp64 = kFp64Too && L.cs.lu_mode == kLu64;
                if (fp64)
                    cell.template factor<double>(s, slot, L.cs.c);
                else
                    cell.template factor<T>(s, slot, L.cs.c);
                if (threadIdx.x == 0) {
                    L.cs.c_lu = L.cs.c;
                    L.cs.lu_valid = 1;
                    L.cs.jv_valid = 1;
                    L.cs.n_lu += 1;
                    if (fp64) L.cs.n_lu64 += 1;
                }
                __syncthreads();
                clk.stop(&t_phase[kPhaseFactor]);
            }
            const int phase = newton_tiny<T, kTiles, kFp64Too>(s, slot, L, y, cell, clk.on ? &t_phase[kPhaseRhs] : nullptr);
            clk.stop(&t_phase[kPhaseNewton]);
            const int mode = L.cs.lu_mode;
            if (rk)
                control_rk<1>(s, L, y, phase, nullptr);
            else
                control_bdf<1>(s, slot, L, y, phase, nullptr);
            if (kF32 && L.cs.lu_mode == kLu64 && mode != kLu64) {
                if (threadIdx.x == 0) atomicAdd(&s.q->n64, 1);
                put_back = kPutBack;
            }
            if (L.cs.status != kRunning) break;
            up = time_up<1>(s, a, t0, L);
            clk.stop(&t_phase[kPhaseControl]);
            if (up || put_back) break;
        }
        store_rows(s, slot, y);
        put_back |= up;
        if (!put_back) finish_slot(s, slot, L.cs, L.cs.status);
        __syncthreads();
        if (threadIdx.x == 0) {
            s.ctl[slot] = L.cs;
            if (put_back)
                hold_slot(s, slot);
            else if (kF32 && L.cs.lu_mode == kLu64)
                atomicAdd(&s.q->n64, -1);
        }
        if (up) break;
    }
    __syncthreads();
    if ((a.flags & kProf) && threadIdx.x < kPhases)
        atomicAdd(&s.q->ticks[threadIdx.x],
                  t_phase[threadIdx.x] - (threadIdx.x == kPhaseNewton ? t_phase[kPhaseRhs] : 0ull));
}

// The narrowest of three widths: the factorisation's accumulators (kTiles^2 tiles
// of 16 x 16) and its unrolled panels decide the kernel's registers; of 4 x 4
// tiles they spill beside the rest, of 2 x 2 they don't.  A solve of one cell of
// 12 species took 13.3 ms with 4 x 4 tiles for every size and takes 11.9 ms.
template <typename T, bool kFp64Too>
static Persistent pick(const DeviceNet &n) {
    const void *fn = n.NP <= 16   ? (const void *)&k_integrate_tiny<T, 1, kFp64Too>
                     : n.NP <= 32 ? (const void *)&k_integrate_tiny<T, 2, kFp64Too>
                                  : (const void *)&k_integrate_tiny<T, 4, kFp64Too>;
    return {fn, 64, TinyLayout<T, kFp64Too>(n).total, kFixedLds<1>, sizeof(T) == sizeof(float) && !kFp64Too};
}

Persistent integrate_tiny(const DeviceNet &n, int prec, bool fp64_too) {
    if (prec != ABDF_PREC_FP32_LU) return pick<double, false>(n);
    return fp64_too ? pick<float, true>(n) : pick<float, false>(n);
}

}  // namespace abdf
