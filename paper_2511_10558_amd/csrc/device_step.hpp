// The step attempts of one cell, carried out by one workgroup of W waves with
// one species per thread (S <= 64 W): starting an attempt, the Newton matrix
// and its factorisation, the corrector, the error test and the step and order
// control, for the BDF and for the ESDIRK.
//
// Integrator: variable-order, variable-step BDF in backward-difference form
// (quasi-constant step size, orders 1..5; the BDF family of paper Sec. 1 in
// the formulation of Shampine & Reichelt 1997, Sec. 2.1-2.3, kappa = 0).
// Per step attempt of a cell:
//   begin   clamp h to land on t_end, predictor x_p = sum_{j<=q} D_j,
//           psi = sum_{j=1..q} gamma_j D_j / gamma_q, c = h / gamma_q
//   factor  when c or the Jacobian changed: form M from J at x_J and factor it
//   newton  <= 4 modified-Newton iterations d <- d + M^{-1}(c f(x) - psi - d)
//   control error test ||d / (q+1)|| <= 1, accept (update differences) or
//           reject (shrink h), order/step selection every q+1 equal steps,
//           Jacobian refresh or h halving on corrector failure.
#pragma once

#include "kernels.hpp"

#include "device_chem.hpp"
#include "device_common.hpp"
#include "device_lu.hpp"
#include "device_lu2.hpp"

#include "../../include/astrobdf.h"

namespace abdf {

// ------------------------------------------------------------ BDF helpers --

__device__ inline double bdf_gamma(int q) {
    double g = 0.0;
    for (int j = 1; j <= q; ++j) g += 1.0 / j;
    return g;
}

__device__ inline double growth(double err, int p) {
    if (err == 0.0) return INFINITY;
    if (!isfinite(err)) return 0.0;
    return pow(err, -1.0 / p);
}

// RU = R(rho) R(1) with R(rho)[i][j] = prod_{m=1..i} (m - 1 - rho j) / m, i, j in 0..q.
// Thread i * 6 + j (< 36) forms entry (i, j): the factors of R(rho)[i][m] and
// R(1)[m][j] in the order of the recurrence R[i][.] = R[i - 1][.] (i - 1 - rho .) / i,
// then the sum over m in order.  Static loop bounds keep everything in registers.
__device__ inline void interp_product(int q, double rho, double *RU) {
    const int t = thread_id();
    if (t >= 36) return;
    const int i = t / 6, j = t % 6;
    if (i > q || j > q) return;
    double s = 0.0;
#pragma unroll
    for (int m = 0; m <= kMaxOrder; ++m) {
        if (m <= q) {
            double rr = 1.0, r1 = 1.0;
#pragma unroll
            for (int k = 1; k <= kMaxOrder; ++k) {
                if (k <= i) rr = rr * (k - 1 - rho * m) / k;
                if (k <= m) r1 = r1 * (k - 1 - 1.0 * j) / k;
            }
            s += rr * r1;
        }
    }
    RU[i * 6 + j] = s;
}

// The conditions of a slot at time t into out[5] (LDS, thread 0): an
// expanding flow, phi_j(t) = phi_j(0) (1 + t / tc)^(-p_j), constant for tc = 0.
__device__ __forceinline__ void phi_at(const Slots &s, int slot, double tc, double t, double *out) {
    if (threadIdx.x == 0) {
        const double *p0 = s.phi + size_t(slot) * 5;
        const double sc = 1.0 + t / tc;
#pragma unroll
        for (int j = 0; j < 5; ++j) out[j] = tc > 0.0 ? p0[j] * pow(sc, -s.phi_exp[j]) : p0[j];
    }
}

// Marks a slot finished and queues it for the harvest (thread 0 writes).
__device__ inline void finish_slot(const Slots &s, int slot, SlotCtl &cs, int status) {
    if (threadIdx.x == 0) {
        cs.status = status;
        const int p = atomicAdd(&s.q->nfin, 1);
        s.fin[p] = slot;
        if (int32_t *host = s.q->fin_host)
            __hip_atomic_store(host + p, slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Queues a running slot for the integration (thread 0 writes).
__device__ inline void queue_slot(const Slots &s, int slot) {
    if (threadIdx.x == 0) {
        const unsigned long long p = atomicAdd(&s.q->tail, 1ull);
        s.fifo[p % unsigned(s.nslots)] = slot;
    }
}

// Takes the next entry of a ring with head counter *head, entries up to limit;
// -1 when none is left.
__device__ inline int take_entry(unsigned long long *head, unsigned long long limit, const int32_t *ring, int n) {
    unsigned long long h = __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (h < limit) {
        const unsigned long long o = atomicCAS(head, h, h + 1);
        if (o == h) return ring[h % unsigned(n)];
        h = o;
    }
    return -1;
}

// Thread 0: the next slot to integrate.  Slots interrupted by the end of the
// last launch come first (those up to held_limit: a slot put back in this
// launch is not taken again before the next), then the admitted ones in order.
__device__ inline int next_slot(const Slots &s, unsigned long long held_limit) {
    const int slot = take_entry(&s.q->held_head, held_limit, s.held, s.nslots);
    return slot >= 0 ? slot : take_entry(&s.q->head, s.q->tail, s.fifo, s.nslots);
}

// Thread 0: puts an interrupted slot back.
__device__ inline void hold_slot(const Slots &s, int slot) {
    const unsigned long long p = atomicAdd(&s.q->held_tail, 1ull);
    s.held[p % unsigned(s.nslots)] = slot;
}

// LDS of a workgroup beside the dynamic block.
template <int W>
struct StepLds {
    SlotCtl cs;
    double RU[36], red[8], phit[5], sh;
    int32_t slot, flag, bad;
};

// Sum over the workgroup, identical on every thread.
template <int W>
__device__ __forceinline__ double wg_sum(double v, double *red) {
    v = wave_sum(v);
    if constexpr (W == 1) return v;
    __syncthreads();
    const int t = thread_id();
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += red[w];
    return s;
}

// Sums of squares over the workgroup, identical on every thread, of N values per
// thread at once.  The order does not depend on the number of waves: species i
// and i + 256 first, then each wave's lanes, then the waves.  fold: 256 N
// doubles of LDS (above 256 species), red: 4 N doubles.
template <int W, int N>
__device__ __forceinline__ void wg_squares(double (&v)[N], int S, double *fold, double *red) {
    const int t = thread_id();
    double a[N];
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = v[k] * v[k];
    if (W > 4 && S > 256) {
        __syncthreads();
        if (t >= 256) {
#pragma unroll
            for (int k = 0; k < N; ++k) fold[256 * k + t - 256] = v[k];
        }
        __syncthreads();
        if (t < 256) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const double o = fold[256 * k + t];
                a[k] = fma(o, o, a[k]);
            }
        }
    }
    constexpr int WR = W > 4 ? 4 : W;
    if (t < 64 * WR) {
#pragma unroll
        for (int k = 0; k < N; ++k) a[k] = wave_sum(a[k]);
    }
    if constexpr (W > 1) {
        __syncthreads();
        if (t < 64 * WR && (t & 63) == 0) {
#pragma unroll
            for (int k = 0; k < N; ++k) red[WR * k + (t >> 6)] = a[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < N; ++k) {
            a[k] = 0.0;
#pragma unroll
            for (int w = 0; w < WR; ++w) a[k] += red[WR * k + w];
        }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = a[k];
}

template <int W>
__device__ __forceinline__ double wg_square(double v, int S, double *fold, double *red) {
    double a[1] = {v};
    wg_squares<W, 1>(a, S, fold, red);
    return a[0];
}

template <int W>
__device__ __forceinline__ bool wg_any(bool p, double *red) {
    return wg_sum<W>(p ? 1.0 : 0.0, red) != 0.0;
}

// What a thread holds of its species during an attempt: the Newton iterate, the
// accumulated correction, psi, the Newton weight, and the rows of the slot's
// difference table (ESDIRK: x_n, F_1, G_2..G_7).
struct SpeciesState {
    double x, d, psi, scl;
    double v[kDRows];
};

__device__ __forceinline__ void load_rows(const Slots &s, int slot, SpeciesState &y) {
    const double *D = s.D + size_t(slot) * kDRows * s.S;
    const int i = thread_id();
#pragma unroll
    for (int j = 0; j < kDRows; ++j) y.v[j] = i < s.S ? D[j * s.S + i] : 0.0;
}

__device__ __forceinline__ void store_rows(const Slots &s, int slot, const SpeciesState &y) {
    double *D = s.D + size_t(slot) * kDRows * s.S;
    const int i = thread_id();
    if (i < s.S) {
#pragma unroll
        for (int j = 0; j < kDRows; ++j) D[j * s.S + i] = y.v[j];
    }
}

// Rows 0..q of the table from spacing h to rho h.  Every row index is static
// (rows above q masked), so that the rows stay in registers.
__device__ __forceinline__ void rescale_rows(SpeciesState &y, int q, double rho, double *RU) {
    __syncthreads();
    interp_product(q, rho, RU);
    __syncthreads();
    double w[kMaxOrder + 1];
#pragma unroll
    for (int a = 0; a <= kMaxOrder; ++a) {
        double sum = 0.0;
#pragma unroll
        for (int b = 0; b <= kMaxOrder; ++b)
            if (b <= q) sum += RU[b * 6 + a] * y.v[b];
        w[a] = sum;
    }
#pragma unroll
    for (int j = 0; j <= kMaxOrder; ++j) y.v[j] = j <= q ? w[j] : y.v[j];
}

// Starts the next step attempt of a running slot (cs in LDS, its rows in y):
// checks limits, lands on t_end and forms the predictor.  With time-dependent
// conditions the slot's rate coefficients become those at the attempt's end,
// t + h.  Leaves cs.status different from kRunning when no attempt can be
// made.  Ends with a barrier.
template <int W>
__device__ __forceinline__ void begin_attempt(const Slots &s, const DeviceNet &n, int slot, StepLds<W> &L,
                                              SpeciesState &y) {
    const int i = thread_id();
    const bool own = i < s.S;
    SlotCtl &cs = L.cs;
    if (threadIdx.x == 0) {
        int st = kRunning;
        double rho = 0.0;
        if (cs.n_attempts >= s.max_steps) {
            st = ABDF_CELL_MAX_STEPS;
        } else {
            cs.n_attempts += 1;
            if (cs.h < 10.0 * kURound * fabs(cs.t)) {
                st = ABDF_CELL_STEP_TOO_SMALL;
            } else {
                cs.landing = 0;
                if (cs.t + cs.h >= cs.t_end) {
                    if (cs.t + cs.h > cs.t_end) {
                        rho = (cs.t_end - cs.t) / cs.h;
                        cs.h = cs.t_end - cs.t;
                        cs.n_equal = 0;
                    }
                    cs.landing = 1;
                }
            }
        }
        cs.status = st;
        L.sh = rho;
    }
    __syncthreads();
    if (cs.status != kRunning) return;
    const int q = cs.q;
    const double rho = L.sh;
    if (rho != 0.0) rescale_rows(y, q, rho, L.RU);
    if (s.tvar && cs.tc > 0.0) {
        phi_at(s, slot, cs.tc, cs.t + cs.h, L.phit);
        __syncthreads();
        cell_rates<64 * W>(n, L.phit, s.k + size_t(slot) * n.R);
    }
    const double gq = bdf_gamma(q);
    const bool refresh = cs.jac_refresh != 0;
    double xp = y.v[0], ps = 0.0;
#pragma unroll
    for (int j = 1; j <= kMaxOrder; ++j)
        if (j <= q) {
            xp = xp + y.v[j];
            ps = ps + bdf_gamma(j) * y.v[j];
        }
    y.x = xp;
    y.d = 0.0;
    y.psi = ps / gq;
    y.scl = own ? atol_of(s, cs, i) + cs.rtol * fabs(xp) : 1.0;
    if (own && refresh) s.xJ[size_t(slot) * s.S + i] = xp;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (refresh) { cs.jac_refresh = 0; cs.lu_valid = 0; cs.jv_valid = 0; }
        cs.c = cs.h / gq;
        const bool stale = s.lu_reuse > 0.0 ? !(fabs(cs.c - cs.c_lu) <= s.lu_reuse * cs.c_lu) : cs.c != cs.c_lu;
        if (stale) cs.lu_valid = 0;
    }
    __syncthreads();
}

// ----------------------------------------------------------------- ESDIRK --
//
// Kvaerno's seven-stage ESDIRK 5(4) (BIT Numer. Math. 44, 2004): explicit
// first stage, diagonal gamma = 0.26, stiffly accurate pair (c_6 = c_7 = 1).
// Stage 2 of an attempt factors I - h gamma J(x_n), stages 3..7 reuse it.  The
// slot's rows hold x_n (0), F_1 = f(x_n) (1) and G_i = h f(Y_i) (2..7).

constexpr int kRkStages = 7;
constexpr double kRkGamma = 0.26;
static __constant__ double kRkA[kRkStages][kRkStages] = {
    {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {0.26, 0.26, 0.0, 0.0, 0.0, 0.0, 0.0},
    {0.13, 0.84033320996790809, 0.26, 0.0, 0.0, 0.0, 0.0},
    {0.22371961478320505, 0.47675532319799699, -0.06470895363112615, 0.26, 0.0, 0.0, 0.0},
    {0.16648564323248321, 0.10450018841591720, 0.03631482272098715, -0.13090704451073998, 0.26, 0.0, 0.0},
    {0.13855640231268224, 0.0, -0.04245337201752043, 0.02446657898003141, 0.61943039072480676, 0.26, 0.0},
    {0.13659751177640291, 0.0, -0.05496908796538376, -0.04118626728321046, 0.62993304899016403,
     0.06962479448202728, 0.26}};

// Starts stage cs.stage (2..7) of a running slot.  Stage 2 opens a step
// attempt: the step budget, the step-size floor and the landing on t_end are
// checked, and after an accepted step the Jacobian point moves to x_n.  The
// stage starts from Y_i^0 = x_n + sum_{j<i} a_ij G_j + gamma G_{i-1} (its own
// equation with the previous stage's G, G_1 = h F_1) with
// psi = Y_i^0 - x_n - sum_{j<i} a_ij G_j and weights atol + rtol |Y_i^0|, so that
// the corrector solves Y_i = x_n + sum_j a_ij G_j + h gamma f(Y_i) as a BDF
// corrector with c = h gamma.  Ends with a barrier.
template <int W>
__device__ __forceinline__ void begin_stage_rk(const Slots &s, int slot, StepLds<W> &L, SpeciesState &y) {
    const int i = thread_id();
    const bool own = i < s.S;
    SlotCtl &cs = L.cs;
    const int stage = cs.stage;
    __syncthreads();
    if (threadIdx.x == 0 && stage == 2) {
        int st = kRunning;
        if (cs.n_attempts >= s.max_steps) {
            st = ABDF_CELL_MAX_STEPS;
        } else {
            cs.n_attempts += 1;
            if (cs.h < 10.0 * kURound * fabs(cs.t)) {
                st = ABDF_CELL_STEP_TOO_SMALL;
            } else {
                cs.landing = 0;
                if (cs.t + cs.h >= cs.t_end) {
                    cs.h = cs.t_end - cs.t;
                    cs.landing = 1;
                }
            }
        }
        cs.status = st;
    }
    __syncthreads();
    if (cs.status != kRunning) return;
    const bool first = stage == 2;
    const bool refresh = first && cs.jac_refresh != 0;
    const double h = cs.h;
    const double *a = kRkA[stage - 1];
    const double xn = y.v[0];
    const double g1 = h * y.v[1];
    double sum = a[0] * g1, gprev = g1;
#pragma unroll
    for (int j = 2; j < kRkStages; ++j)
        if (j < stage) {
            sum = sum + a[j - 1] * y.v[j];
            gprev = y.v[j];
        }
    const double xp = (xn + sum) + kRkGamma * gprev;
    y.x = xp;
    y.d = 0.0;
    y.psi = (xp - xn) - sum;
    y.scl = own ? atol_of(s, cs, i) + cs.rtol * fabs(xp) : 1.0;
    if (own && refresh) s.xJ[size_t(slot) * s.S + i] = xn;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double c = h * kRkGamma;
        if (refresh) {
            cs.jac_refresh = 0;
            cs.jv_valid = 0;
            cs.lu_valid = 0;
            cs.n_jac += 1;
        }
        if (first && c != cs.c_lu) cs.lu_valid = 0;
        cs.c = c;
    }
    __syncthreads();
}

// ----------------------------------------------------------------- factor --

// Forms M = I - c J(x_J) of a slot and factors it in T.  x_J is staged in LDS
// where the factorisation's own data go afterwards; the Jacobian nonzeros go to
// the slot's compact array and M is formed block column by block column as
// the factorisation gathers it.  A factorisation for a new c at the same x_J
// (modified Newton keeps J across steps) reuses the nonzeros already there.
template <typename T, int W>
__device__ __forceinline__ void factor_slot(const Slots &s, const DeviceNet &n, int slot, const SlotCtl &cs,
                                            double *smem) {
    const int S = s.S, NP = s.NP;
    double *jv = s.jval + size_t(slot) * n.nnzJ;
    if (!cs.jv_valid) {
        // x_J and the rate coefficients, which the terms read at random, in LDS
        const double *k = s.k + size_t(slot) * n.R;
        const int i = thread_id();
        if (i < S) smem[i] = s.xJ[size_t(slot) * S + i];
        for (int r = i; r < n.R; r += 64 * W) smem[S + r] = k[r];
        __syncthreads();
        jacobian_values<64 * W>(n, smem + S, smem, jv);
        __syncthreads();
    }
    NewtonMatrixSource<T> src{n.jmask, n.jbase, n.nbw, jv, uniform(cs.c)};
    lu_factor_left<T, W, 4>(SlotStorage<T>{slot_lu<T>(s, slot), s.lda}, NP, s.perm + size_t(slot) * NP, slot_dinv<T>(s, slot), nullptr,
                         reinterpret_cast<unsigned char *>(smem), src);
    __syncthreads();
}

// ----------------------------------------------------------------- newton --

// z = M^{-1} b with the slot's factors (b, z in LDS [NP]; scratch: 64 doubles and
// NP row indices).  Ends with a barrier.
template <typename T, int W>
__device__ __forceinline__ void solve_slot(const Slots &s, int slot, const double *b, double *z, double *scratch) {
    const int S = s.S, NP = s.NP, tid = thread_id();
    int32_t *perm = reinterpret_cast<int32_t *>(scratch + kLuW);
    if (tid < NP) perm[tid] = s.perm[size_t(slot) * NP + tid];
    __syncthreads();
    const int N = min(NP, S + (S & 1));   // the padding past S is the identity's
    // FP64: 6 tiles of 16 registers a thread in flight
    constexpr int kDepth = sizeof(T) == sizeof(double) ? 6 : 8;
    lu_solve_left<T, 64 * W, kDepth>(slot_lu<T>(s, slot), s.lda, slot_dinv<T>(s, slot), perm, NP, N, b, z,
                                     scratch);
}

// The convergence and divergence tests after Newton iteration m with correction
// norm eta (the previous one eta_old).
__device__ __forceinline__ int newton_verdict(double eta, double eta_old, int m, int maxiter, double tol) {
    bool fail = false, conv = false;
    double theta = -1.0;
    if (m > 1) {
        theta = eta / eta_old;
        // theta^(maxiter - m), the power by repeated products
        double pw = 1.0;
        for (int e = maxiter - m; e > 0; --e) pw *= theta;
        fail = theta >= 1.0 || pw / (1.0 - theta) * eta > tol;
    }
    if (!fail) conv = eta == 0.0 || (m > 1 && theta / (1.0 - theta) * eta < tol);
    if (!fail && !conv && m == maxiter) fail = true;
    return fail ? kFailed : (conv ? kConverged : kIter);
}

// The corrector of one attempt: residual r = c f(x) - psi - d, correction
// Delta = M^{-1} r, its weighted norm, the convergence and divergence tests,
// x += Delta, d += Delta.  A non-finite f ends the attempt as a corrector
// failure.  Returns kConverged or kFailed; the counters of cs are updated.
// FP32-LU cells after a corrector failure refine each solve once in FP64:
// Delta += M^{-1} (r - (Delta - c J(x_J) Delta)), J applied through the
// reactions.  LDS: b, z [NP] each (refining: z2 [NP]), xs [S], rate [R] (the
// solves' scratch shares rate's place).  Ends with a barrier.
template <int W, bool kF32>
__device__ __forceinline__ int newton_slot(const Slots &s, const DeviceNet &n, int slot, StepLds<W> &L,
                                           SpeciesState &y, double *smem, unsigned long long *t_rhs) {
    constexpr int NT = 64 * W;
    const int S = s.S, NP = s.NP, i = thread_id();
    const bool own = i < S;
    SlotCtl &cs = L.cs;
    double *b = smem, *z = b + NP, *z2 = z + NP;
    double *xs = kF32 ? z2 + NP : z2, *rate = xs + S;
    const double *k = s.k + size_t(slot) * n.R;
    const double c = uniform(cs.c), c_lu = uniform(cs.c_lu), tol = uniform(cs.newton_tol);
    const int mode = kF32 ? __builtin_amdgcn_readfirstlane(cs.lu_mode) : kLu64;
    double eta_old = 0.0;
    int phase = kIter, m = 0;
    while (phase == kIter) {
        ++m;
        const unsigned long long t0 = t_rhs && i == 0 ? wall_clock64() : 0ull;
        if (own) xs[i] = y.x;
        if (i == 0) L.bad = 0;
        __syncthreads();
        cell_rhs_ahead<NT>(n, k, xs, rate, b);
        double r = 0.0;
        if (own) {
            const double f = b[i];
            r = c * f - y.psi - y.d;
            if (!isfinite(f)) L.bad = 1;
        }
        if (i < NP) b[i] = r;
        __syncthreads();
        if (t_rhs && i == 0) *t_rhs += wall_clock64() - t0;
        if (L.bad) {
            phase = kFailed;
            break;
        }
        if (kF32 && mode != kLu64)
            solve_slot<float, W>(s, slot, b, z, rate);
        else
            solve_slot<double, W>(s, slot, b, z, rate);
        if (kF32 && mode == kLuRefined32) {
            if (own) xs[i] = s.xJ[size_t(slot) * S + i];
            __syncthreads();
            cell_jvp<NT>(n, k, xs, z, rate, z2);   // z2 = J(x_J) z
            if (i < NP) b[i] = own ? r - (z[i] - c_lu * z2[i]) : 0.0;
            __syncthreads();
            solve_slot<float, W>(s, slot, b, z2, rate);
            if (i < NP) z[i] = z[i] + z2[i];
        }
        double delta = own ? z[i] : 0.0;
        // a factorisation kept from c_lu != c: the correction is scaled by
        // 2 / (1 + c / c_lu), the usual remedy for the lagged leading coefficient
        if (c != c_lu) delta = delta * (2.0 / (1.0 + c / c_lu));
        const double eta = sqrt(wg_square<W>(delta / y.scl, S, rate, L.red) / S);
        const int verdict = newton_verdict(eta, eta_old, m, s.newton_maxiter, tol);
        eta_old = eta;
        // a failed attempt discards x and d
        if (verdict != kFailed) {
            y.x = y.x + delta;
            y.d = y.d + delta;
        }
        phase = verdict;
    }
    if (i == 0) {
        cs.n_rhs += m;
        cs.n_newton_iter += m;
        cs.m_last = m;
    }
    __syncthreads();
    return phase;
}

// ---------------------------------------------------------------- control --

// Acts on the outcome of a BDF attempt (y.v: the slot's rows 0..q+2 on entry,
// updated on return): cs becomes the state the next attempt starts from, or
// its status leaves kRunning.  Ends with a barrier.
template <int W>
__device__ __forceinline__ void control_bdf(const Slots &s, int slot, StepLds<W> &L, SpeciesState &y, int phase,
                                            double *smem) {
    const int i = thread_id(), S = s.S;
    const bool own = i < S;
    SlotCtl &cs = L.cs;
    const int q = cs.q;
    if (phase == kFailed) {
        if (i == 0) {
            cs.n_newton_fail += 1;
            L.sh = 0.0;
            if (!cs.j_fresh) {
                cs.j_fresh = 1;
                cs.jac_refresh = 1;
                cs.n_jac += 1;
            } else if (s.lu_reuse > 0.0 && cs.c != cs.c_lu) {
                // fresh Jacobian, factorisation kept from another c: retry the
                // same step with the factorisation at the current c
                cs.lu_valid = 0;
            } else if (s.prec == ABDF_PREC_FP32_LU && cs.lu_mode != kLu64) {
                // the corrector failed with a fresh Jacobian and FP32 factors:
                // the cell retries the same step with refined solves, then
                // with FP64 factors
                cs.lu_mode += 1;
                if (cs.lu_mode == kLu64) cs.lu_valid = 0;
            } else {
                cs.h = 0.5 * cs.h;
                cs.n_equal = 0;
                if (s.lu_reuse == 0.0) cs.lu_valid = 0;   // else the change of c decides
                L.sh = 0.5;
            }
        }
        __syncthreads();
        if (L.sh != 0.0) rescale_rows(y, q, 0.5, L.RU);
        __syncthreads();
        return;
    }
    // converged: local error test
    const double rtol = cs.rtol;
    const double eq = 1.0 / (q + 1);
    const double sc = own ? atol_of(s, cs, i) + rtol * fmax(fabs(y.v[0]), fabs(y.x)) : 1.0;
    const double err = sqrt(wg_square<W>(own ? eq * y.d / sc : 0.0, S, smem, L.red) / S);
    const int m = cs.m_last;
    const double safety = 0.9 * (2 * kNewtonMaxIter + 1) / (2 * kNewtonMaxIter + m);
    if (!isfinite(err)) {
        __syncthreads();
        if (i == 0) cs.status = ABDF_CELL_NONFINITE;
        __syncthreads();
        return;
    }
    if (err > 1.0) {
        const double rho = fmax(kMinFactor, safety * growth(err, q + 1));
        __syncthreads();
        if (i == 0) {
            cs.n_err_reject += 1;
            cs.h = cs.h * rho;
            cs.n_equal = 0;
            if (s.lu_reuse == 0.0) cs.lu_valid = 0;   // else the change of c decides
        }
        rescale_rows(y, q, rho, L.RU);
        __syncthreads();
        return;
    }
    // accept: update the differences, collect the order-selection norms, and
    // record the step when a tape is attached and the step is in the cell's window
    const int rel = cs.n_steps - (s.tape_w0 ? s.tape_w0[cs.cell] : 0);
    if (s.tape_x && rel >= s.tape_cap && !s.tape_overflow) {
        __syncthreads();
        if (i == 0) cs.status = ABDF_CELL_TAPE_FULL;
        __syncthreads();
        return;
    }
    const size_t te = size_t(cs.cell) * s.tape_cap + rel;
    double *tx = s.tape_x && rel >= 0 && rel < s.tape_cap ? s.tape_x + te * S : nullptr;
    const double em_c = q > 1 ? 1.0 / q : 0.0;
    const double ep_c = 1.0 / (q + 2);
    // rows 0..q+2 of the difference table, with every index static (masks and
    // selects instead of v[q + 1] etc.) so that v stays in registers
    double *v = y.v;
    double vq1 = 0.0;
#pragma unroll
    for (int j = 0; j < kDRows; ++j) vq1 = j == q + 1 ? v[j] : vq1;
#pragma unroll
    for (int j = 0; j < kDRows; ++j) {
        if (j == q + 2) v[j] = y.d - vq1;
        if (j == q + 1) v[j] = y.d;
    }
#pragma unroll
    for (int j = kDRows - 2; j >= 0; --j)
        if (j <= q) v[j] = v[j] + v[j + 1];
    if (tx && own) tx[i] = v[0];
    double vq = 0.0, vq2 = 0.0;
#pragma unroll
    for (int j = 0; j < kDRows; ++j) {
        vq = j == q ? v[j] : vq;
        vq2 = j == q + 2 ? v[j] : vq2;
    }
    const double a1 = em_c * vq / sc, a2 = ep_c * vq2 / sc;
    double sums[2] = {own ? a1 : 0.0, own ? a2 : 0.0};
    if (i == 0) L.bad = 0;
    wg_squares<W, 2>(sums, S, smem, L.red);
    const double sm = sums[0], sp = sums[1];
    if constexpr (W == 1) __syncthreads();
    if (own && !isfinite(v[0])) L.bad = 1;
    if (i == 0) {
        if (tx) {
            s.tape_h[te] = cs.h;
            s.tape_q[te] = q;
        } else if (s.tape_x && rel == -1 && s.tape_hprev) {
            s.tape_hprev[cs.cell] = cs.h;
            s.tape_qprev[cs.cell] = q;
        }
        cs.t = cs.landing ? cs.t_end : cs.t + cs.h;
        cs.n_steps += 1;
        cs.n_equal += 1;
        cs.j_fresh = 0;
    }
    __syncthreads();
    if (L.bad || cs.landing || (s.tape_stop && cs.n_steps >= s.tape_stop[cs.cell])) {
        // not finite, t_end reached, or a re-run has recorded its window
        const int st = L.bad ? ABDF_CELL_NONFINITE : ABDF_CELL_OK;
        __syncthreads();
        if (i == 0) cs.status = st;
        __syncthreads();
        return;
    }
    if (cs.n_equal >= q + 1) {
        __syncthreads();
        if (i == 0) {
            const double e_m = q > 1 ? sqrt(sm / S) : INFINITY;
            const double e_p = q < s.max_order ? sqrt(sp / S) : INFINITY;
            const double r0 = growth(e_m, q), r1 = growth(err, q + 1), r2 = growth(e_p, q + 2);
            int best = 1;
            double rb = r1;
            if (r0 > rb) { best = 0; rb = r0; }
            if (r2 > rb) { best = 2; rb = r2; }
            cs.q = q + best - 1;
            double rho = fmin(kMaxFactor, safety * rb);
            if (s.h_max > 0.0) rho = fmin(rho, s.h_max / cs.h);
            cs.h = cs.h * rho;
            cs.n_equal = 0;
            if (s.lu_reuse == 0.0) cs.lu_valid = 0;   // else the change of c decides
            L.sh = rho;
        }
        __syncthreads();
        const double rho = L.sh;
        rescale_rows(y, cs.q, rho, L.RU);
    }
    __syncthreads();
}

// Acts on the ESDIRK stage just solved: a converged stage stores
// G_i = (psi + d) / gamma (its own equation gives h f(Y_i)); after stage 7 the
// error test Y_7 - Y_6 decides the step.  Ends with a barrier.
template <int W>
__device__ __forceinline__ void control_rk(const Slots &s, StepLds<W> &L, SpeciesState &y, int phase, double *smem) {
    const int i = thread_id(), S = s.S;
    const bool own = i < S;
    SlotCtl &cs = L.cs;
    const int stage = cs.stage;
    __syncthreads();
    if (phase == kFailed) {
        if (i == 0) {
            cs.n_newton_fail += 1;
            if (s.prec == ABDF_PREC_FP32_LU && cs.lu_mode != kLu64) {
                // FP32 factors: the same step again with refined solves, then
                // with FP64 factors
                cs.lu_mode += 1;
                if (cs.lu_mode == kLu64) cs.lu_valid = 0;
            } else {
                cs.h = 0.5 * cs.h;
                cs.rejected = 1;
            }
            cs.stage = 2;
        }
        __syncthreads();
        return;
    }
    const double gi = (y.psi + y.d) / kRkGamma;
#pragma unroll
    for (int j = 2; j <= kRkStages; ++j)
        if (j == stage) y.v[j] = gi;
    if (stage < kRkStages) {
        if (i == 0) cs.stage = stage + 1;
        __syncthreads();
        return;
    }
    // error estimate Y_7 - Y_6 = sum_j (a_7j - a_6j) G_j, weights from x_n and Y_7
    const double h = cs.h, rtol = cs.rtol;
    double ev = 0.0;
    if (own) {
        double e = (kRkA[6][0] - kRkA[5][0]) * (h * y.v[1]);
#pragma unroll
        for (int j = 2; j <= kRkStages; ++j) e = e + (kRkA[6][j - 1] - kRkA[5][j - 1]) * y.v[j];
        const double sc = atol_of(s, cs, i) + rtol * fmax(fabs(y.v[0]), fabs(y.x));
        ev = e / sc;
    }
    const double err = sqrt(wg_square<W>(ev, S, smem, L.red) / S);
    if (!isfinite(err)) {
        __syncthreads();
        if (i == 0) cs.status = ABDF_CELL_NONFINITE;
        __syncthreads();
        return;
    }
    if (err > 1.0) {
        __syncthreads();
        if (i == 0) {
            cs.n_err_reject += 1;
            cs.h = cs.h * fmax(kMinFactor, 0.9 * pow(err, -0.2));
            cs.rejected = 1;
            cs.stage = 2;
        }
        __syncthreads();
        return;
    }
    // accept: x_{n+1} = Y_7, and F_1 of the next step is G_7 / h
    y.v[0] = y.x;
    y.v[1] = y.v[kRkStages] / h;
    const bool nonfinite = wg_any<W>(own && !isfinite(y.x), L.red);
    __syncthreads();
    if (i == 0) {
        cs.t = cs.landing ? cs.t_end : cs.t + h;
        cs.n_steps += 1;
        cs.jac_refresh = 1;
        if (nonfinite || cs.landing) {
            cs.status = nonfinite ? ABDF_CELL_NONFINITE : ABDF_CELL_OK;
        } else {
            double fac = err == 0.0 ? kMaxFactor : fmin(kMaxFactor, fmax(kMinFactor, 0.9 * pow(err, -0.2)));
            if (cs.rejected) {
                fac = fmin(1.0, fac);
                cs.rejected = 0;
            }
            cs.h = h * fac;
            if (s.h_max > 0.0) cs.h = fmin(cs.h, s.h_max);
            cs.stage = 2;
        }
    }
    __syncthreads();
}

}  // namespace abdf
