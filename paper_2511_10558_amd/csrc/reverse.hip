// The discrete adjoint's reverse sweep.
#include "integrate_kernels.hpp"

namespace abdf {

// ---------------------------------------------------------------- adjoint --
//
// Reverse sweep of the frozen-sequence BDF map: the accepted (h_n, q_n) of a
// recorded solve, each corrector equation c f(x_{n+1}) - psi - d = 0 taken as
// solved exactly.  lambda_j (stored in D) is the adjoint of difference row j.
// Step n, in reverse:
//   difference update   lambda_{j+1} += lambda_j (j = 0..q), lambda_d =
//                       lambda_{q+1} + lambda_{q+2}, lambda_{q+1} = -lambda_{q+2},
//                       lambda_{q+2} = 0
//   corrector           mu = M^{-T} lambda_d with M = I - c J(x_{n+1}) factored afresh,
//                       solved as lambda_xp = mu - lambda_d = M^{-T} c J^T lambda_d
//   predictor           lambda_j += lambda_xp (j <= q), lambda_j -= gamma_j / gamma_q mu (1 <= j <= q)
//   parameters          dL/dk_r += c x_a x_b (nu_r . mu)   (x at x_{n+1}, x_b only for two reactants)
//   step-size change    lambda_{0..q} <- (R(rho) U) lambda when (h, q) changed from step n-1
// and finally, for D_0 = x_0 and D_1 = h_0 f(x_0):
//   dL/dk_r += h_0 x_a x_b (nu_r . lambda_1) at x_0,  dL/dx_0 = lambda_0 + h_0 J(x_0)^T lambda_1.
// The sweep accumulates the gradient with respect to the rate coefficients;
// dL/dlog alpha_r = k_r dL/dk_r (k_r is linear in alpha_r) and the gradient with
// respect to a cell's physical parameters, sum_r dL/dk_r dk_r/dphi, are formed
// when the cell finishes.  Neither divides by a parameter, so both stay finite
// where G0 = 0 or zeta = 0 switches a family of reactions off.

// x_a (x_b): the abundance factor of rate_r = k_r x_a (x_b), from the packed reactant pair
__device__ __forceinline__ double reactant_product(const DeviceNet &n, const double *xs, int r) {
    const int ab = n.rx_ab[r];
    const int a = ab & 0xffff, b = (ab >> 16) & 0xffff;
    double v = xs[a];
    if (b != 0xffff) v *= xs[b];
    return v;
}

// nu_r . v over the reaction's net stoichiometry
__device__ __forceinline__ double nu_dot(const DeviceNet &n, const double *v, int r) {
    double w = 0.0;
    for (int e = n.rnu_ptr[r]; e < n.rnu_ptr[r + 1]; ++e) {
        const int ent = n.rnu_ent[e];
        w += double((ent & 7) - 4) * v[ent >> 3];
    }
    return w;
}

// Reverse of rescale_D: lambda_old[b] = sum_a RU[b][a] lambda_new[a], rows 0..q.
template <int NT>
__device__ __forceinline__ void rescale_adjoint(double *L, int S, int q, double rho, double *RU) {
    interp_product(q, rho, RU);
    __syncthreads();
    for (int i = thread_id(); i < S; i += NT) {
        double v[kMaxOrder + 1], w[kMaxOrder + 1];
#pragma unroll
        for (int j = 0; j <= kMaxOrder; ++j) v[j] = j <= q ? L[j * S + i] : 0.0;
#pragma unroll
        for (int b = 0; b <= kMaxOrder; ++b) {
            double acc = 0.0;
#pragma unroll
            for (int a = 0; a <= kMaxOrder; ++a)
                if (a <= q) acc += RU[b * 6 + a] * v[a];
            w[b] = acc;
        }
#pragma unroll
        for (int j = 0; j <= kMaxOrder; ++j)
            if (j <= q) L[j * S + i] = w[j];
    }
    __syncthreads();
}

// c J(x)^T v (into out, global) for one slot: w_r = nu_r . v, then
// (J^T v)_j = sum over reactions r with reactant j of d rate_r / d x_j w_r.
// xs, v in LDS; w: LDS scratch [R].
template <int NT>
__device__ __forceinline__ void jac_transpose_apply(const DeviceNet &n, const double *k, const double *xs,
                                                    const double *v, double *w, double c, double *out, int S) {
    for (int r = thread_id(); r < n.R; r += NT) w[r] = nu_dot(n, v, r);
    __syncthreads();
    for (int j = thread_id(); j < S; j += NT) {
        double jt = 0.0;
        for (int e = n.dcol_ptr[j]; e < n.dcol_ptr[j + 1]; ++e) {
            const int ent = n.dcol_ent[e];
            const int r = ent >> 16, o = (ent & 0xffff) - 1;
            double d = n.dcol_coef[e] * k[r];
            if (o >= 0) d *= xs[o];
            jt += d * w[r];
        }
        out[j] = c * jt;
    }
    __syncthreads();
}

// Starts reverse step cs.n_steps - 1 of a slot: the reverse of its difference
// update (lambda_d kept in psi), the corrector point, c, and the right-hand
// side c J(x_{n+1})^T lambda_d of the transposed solve.  The solve then
// yields lambda_xp = mu - lambda_d = M^{-T} c J^T lambda_d directly: the
// adjoint rows can be many orders of magnitude larger than lambda_xp, and
// forming mu first and subtracting lambda_d would lose it to cancellation.
// LDS: xs [S], ls [S], w [R].
template <int NT>
__device__ __forceinline__ void adj_begin(const Slots &s, const DeviceNet &n, int slot, SlotCtl &cs, double *smem) {
    const int S = s.S;
    const int w0 = s.tape_w0 ? s.tape_w0[cs.cell] : 0;
    const size_t te = size_t(cs.cell) * s.tape_cap + (cs.n_steps - 1 - w0);
    const int q = s.tape_q[te];
    const double h = s.tape_h[te];
    const double c = h / bdf_gamma(q);
    double *L = s.D + size_t(slot) * kDRows * S;
    double *rb = s.rb + size_t(slot) * S, *xJ = s.xJ + size_t(slot) * S, *lam_d = s.psi + size_t(slot) * S;
    const double *xt = s.tape_x + te * S;
    double *xs = smem, *ls = xs + S, *w = ls + S;
    for (int i = thread_id(); i < S; i += NT) {
        double v[kDRows];
        for (int j = 0; j <= q + 2; ++j) v[j] = L[j * S + i];
        for (int j = 0; j <= q; ++j) v[j + 1] = v[j + 1] + v[j];
        const double ld = v[q + 1] + v[q + 2];
        v[q + 1] = -v[q + 2];
        v[q + 2] = 0.0;
        for (int j = 0; j <= q + 2; ++j) L[j * S + i] = v[j];
        ls[i] = ld;
        lam_d[i] = ld;
        const double xv = xt[i];
        xs[i] = xv;
        xJ[i] = xv;
    }
    __syncthreads();
    jac_transpose_apply<NT>(n, s.k + size_t(slot) * n.R, xs, ls, w, c, rb, S);
    if (threadIdx.x == 0) {
        cs.h = h;
        cs.q = q;
        cs.c = c;
        cs.jv_valid = 0;   // x_J moved to the step's corrector point
    }
    __syncthreads();
}

// Contributions of the starting differences and dL/dx_0 (into s.x); ends the slot.
// LDS: xs [S], l1 [S], w [R].
template <int NT>
__device__ __forceinline__ void adj_finish(const Slots &s, const DeviceNet &n, int slot, SlotCtl &cs, int len,
                                           double *smem) {
    const int S = s.S, R = n.R;
    double *L = s.D + size_t(slot) * kDRows * S;
    double *dx0 = s.x + size_t(slot) * S;
    if (len > 0) {
        double *xs = smem, *l1 = xs + S, *w = l1 + S;
        const double h0 = s.tape_h[size_t(cs.cell) * s.tape_cap];
        const double *x0 = s.tape_x0 + size_t(cs.cell) * S;
        const double *k = s.k + size_t(slot) * R;
        double *g = s.g + size_t(slot) * R;
        for (int i = thread_id(); i < S; i += NT) {
            xs[i] = x0[i];
            l1[i] = L[S + i];
        }
        __syncthreads();
        for (int r = thread_id(); r < R; r += NT) g[r] += h0 * reactant_product(n, xs, r) * nu_dot(n, l1, r);
        __syncthreads();
        // dL/dx0 = lambda_0 + h0 J(x0)^T lambda_1 (dx0 first holds the second term)
        jac_transpose_apply<NT>(n, k, xs, l1, w, h0, dx0, S);
        for (int i = thread_id(); i < S; i += NT) dx0[i] = L[i] + dx0[i];
    } else {
        for (int i = thread_id(); i < S; i += NT) dx0[i] = L[i];
    }
    __syncthreads();
    finish_slot(s, slot, cs, cs.status == kRunning ? ABDF_CELL_OK : cs.status);
    __syncthreads();
    if (threadIdx.x == 0) s.ctl[slot] = cs;
}

// Completes the current reverse step of a slot: the corrector's and the
// predictor's adjoint, the gradient of its rate coefficients, the reverse of
// the step-size change before it.  Leaves cs.n_steps at the steps still to
// sweep.  Ends with a barrier.
template <int NT>
__device__ __forceinline__ void adj_step(const Slots &s, const DeviceNet &n, int slot, SlotCtl &cs, double *smem,
                                         double *RU) {
    const int S = s.S, R = n.R;
    const int q = cs.q;
    const double c = cs.c, gq = bdf_gamma(q);
    double *L = s.D + size_t(slot) * kDRows * S;
    const double *lam_d = s.psi + size_t(slot) * S, *lxp_g = s.d + size_t(slot) * S, *xJ = s.xJ + size_t(slot) * S;
    double *xs = smem, *ms = xs + S;
    double gr[kMaxOrder + 1];
    for (int j = 1; j <= q; ++j) gr[j] = bdf_gamma(j) / gq;
    for (int i = thread_id(); i < S; i += NT) {
        const double lxp = lxp_g[i];
        const double m = lam_d[i] + lxp;
        xs[i] = xJ[i];
        ms[i] = m;
        L[i] = L[i] + lxp;
        for (int j = 1; j <= q; ++j) L[j * S + i] = L[j * S + i] + (lxp - gr[j] * m);
    }
    __syncthreads();
    double *g = s.g + size_t(slot) * R;
    for (int r = thread_id(); r < R; r += NT) g[r] += c * reactant_product(n, xs, r) * nu_dot(n, ms, r);
    __syncthreads();
    const int m = cs.n_steps - 1;
    const int w0 = s.tape_w0 ? s.tape_w0[cs.cell] : 0;
    if (m > 0) {
        // (h, q) of step m - 1: in the window, or the one recorded just before it
        const size_t te = size_t(cs.cell) * s.tape_cap + (m - 1 - w0);
        const double hp = m > w0 ? s.tape_h[te] : s.tape_hprev[cs.cell];
        const int qp = m > w0 ? s.tape_q[te] : s.tape_qprev[cs.cell];
        if (cs.h != hp || q != qp) rescale_adjoint<NT>(L, S, q, cs.h / hp, RU);
    }
    if (threadIdx.x == 0) cs.n_steps = m;
    __syncthreads();
}

// Places cells in slots for the reverse sweep: lambda_0 = dL/dx(t_end), rate
// coefficients, zero gradient, and the slot queued.
__global__ void __launch_bounds__(kBlock) k_adj_admit(Slots s, DeviceNet n, AdjArgs a) {
    extern __shared__ double smem[];
    __shared__ SlotCtl cs;
    const int idx = blockIdx.x;
    if (idx >= a.count) return;
    const int slot = a.slots[idx];
    const long long cell = a.cells[idx];
    const int S = s.S, R = n.R;
    const bool ok = a.status[cell] == ABDF_CELL_OK;
    if (s.win_end && s.win_end[cell] < 0) {
        // windowed sweep: nothing of this cell in the pass
        if (threadIdx.x == 0) {
            SlotCtl z = {};
            z.cell = int32_t(cell);
            cs = z;
        }
        __syncthreads();
        finish_slot(s, slot, cs, kSitsOut);
        __syncthreads();
        if (threadIdx.x == 0) s.ctl[slot] = cs;
        return;
    }
    double *phi = s.phi + size_t(slot) * 5;
    if (threadIdx.x == 0) {
        for (int j = 0; j < 5; ++j) phi[j] = a.phi[cell * 5 + j];
        SlotCtl z = {};
        z.cell = int32_t(cell);
        z.n_steps = ok ? (s.win_end ? s.win_end[cell] : s.tape_len[cell]) : 0;
        z.status = ok ? kRunning : a.status[cell];
        z.q = 1;
        cs = z;
    }
    double *L = s.D + size_t(slot) * kDRows * S;
    double *g = s.g + size_t(slot) * R;
    if (ok && s.win_resume) {
        // the adjoint rows and dL/dk where the previous pass (the later window) left them
        const double *wl = s.win_lam + size_t(cell) * kDRows * S;
        for (int i = thread_id(); i < kDRows * S; i += kBlock) L[i] = wl[i];
        for (int r = thread_id(); r < R; r += kBlock) g[r] = s.win_g[size_t(cell) * R + r];
    } else {
        for (int i = thread_id(); i < S; i += kBlock) {
            L[i] = ok ? a.dLdx[cell * S + i] : 0.0;
            for (int j = 1; j < kDRows; ++j) L[j * S + i] = 0.0;
        }
        for (int r = thread_id(); r < R; r += kBlock) g[r] = 0.0;
    }
    __syncthreads();
    cell_rates(n, phi, s.k + size_t(slot) * R);
    __syncthreads();
    if (cs.n_steps == 0) {
        adj_finish<kBlock>(s, n, slot, cs, 0, smem);
        return;
    }
    if (threadIdx.x == 0) s.ctl[slot] = cs;
    queue_slot(s, slot);
}

// Sweeps the recorded steps of queued cells backwards, one cell per workgroup.
template <int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2)))
k_reverse(Slots s, DeviceNet n, IntegrateArgs a) {
    constexpr int NT = 64 * W;
    extern __shared__ double smem[];
    __shared__ StepLds<W> L;
    __shared__ unsigned long long t_phase[kPhases];
    const unsigned long long t0 = wall_clock64();
    if (threadIdx.x < kPhases) t_phase[threadIdx.x] = 0;
    PhaseClock clk{(a.flags & kProf) && threadIdx.x == 0, 0};
    const int S = s.S, R = n.R, NP = s.NP;
    while (true) {
        const int slot = take_slot<W>(s, a, L);
        if (slot < 0) break;
        SlotCtl &cs = L.cs;
        const int w0 = s.tape_w0 ? s.tape_w0[cs.cell] : 0;
        bool up = false;
        while (true) {
            clk.start();
            adj_begin<NT>(s, n, slot, cs, smem);
            clk.stop(&t_phase[kPhaseAdjStep]);
            factor_slot<double, W>(s, n, slot, cs, smem);
            if (threadIdx.x == 0) {
                cs.jv_valid = 1;
                cs.n_lu += 1;
            }
            clk.stop(&t_phase[kPhaseFactor]);
            {
                // lambda_xp = M^{-T} (c J^T lambda_d)
                double *b = smem, *z = b + NP, *t = z + NP, *Db = t + (1 + W) * kLuW;
                const double *rb = s.rb + size_t(slot) * S;
                for (int i = thread_id(); i < NP; i += NT) b[i] = i < S ? rb[i] : 0.0;
                __syncthreads();
                lu_solve_left_T<double, W>(slot_lu<double>(s, slot), s.lda, s.perm + size_t(slot) * NP, NP, b, z, t, Db);
                double *d = s.d + size_t(slot) * S;
                for (int i = thread_id(); i < S; i += NT) d[i] = z[i];
                __syncthreads();
            }
            clk.stop(&t_phase[kPhaseAdjSolve]);
            adj_step<NT>(s, n, slot, cs, smem, L.RU);
            if (cs.n_steps <= w0) break;
            up = time_up<W>(s, a, t0, L);
            clk.stop(&t_phase[kPhaseAdjStep]);
            if (up) break;
        }
        if (up) {
            if (threadIdx.x == 0) {
                s.ctl[slot] = cs;
                hold_slot(s, slot);
            }
            break;
        }
        if (cs.n_steps > 0) {
            // the window is swept: the earlier steps come in the next pass
            const double *lam = s.D + size_t(slot) * kDRows * S, *g = s.g + size_t(slot) * R;
            double *wl = s.win_lam + size_t(cs.cell) * kDRows * S;
            for (int i = thread_id(); i < kDRows * S; i += NT) wl[i] = lam[i];
            for (int r = thread_id(); r < R; r += NT) s.win_g[size_t(cs.cell) * R + r] = g[r];
            __syncthreads();
            finish_slot(s, slot, cs, kWindowDone);
            __syncthreads();
            if (threadIdx.x == 0) s.ctl[slot] = cs;
        } else {
            adj_finish<NT>(s, n, slot, cs, 1, smem);
        }
        clk.stop(&t_phase[kPhaseAdjStep]);
    }
    __syncthreads();
    if ((a.flags & kProf) && threadIdx.x < kPhases) atomicAdd(&s.q->ticks[threadIdx.x], t_phase[threadIdx.x]);
}

Persistent reverse_kernel(const DeviceNet &n) {
    constexpr int W = kIntegrateWaves;
    const size_t solve = sizeof(double) * (2 * size_t(n.NP) + (1 + W) * kLuW + kLuW * kLdb);
    const size_t step = sizeof(double) * (2 * size_t(n.S) + n.R);
    return {(const void *)&k_reverse<W>, 64 * W, std::max({lu2_lds_bytes<double, W>(n.NP), solve, step}), kFixedLds<W>};
}

hipError_t launch_adj_admit(const Slots &s, const DeviceNet &n, const AdjArgs &a, size_t lds, hipStream_t st) {
    if (a.count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_adj_admit, dim3(a.count), dim3(kBlock), lds, st, s, n, a);
    return hipGetLastError();
}

}  // namespace abdf
