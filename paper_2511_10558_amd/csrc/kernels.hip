// Admission and harvest of cells, and the kernels of the component entry
// points.  The integration itself is in integrate.hip.
//
// One workgroup handles one cell (slot) in every per-cell kernel; vectors are
// slot-major so a workgroup's loads over species or reactions are coalesced.
#include "device_step.hpp"

namespace abdf {

// --------------------------------------------------------------- kernels --

// Admits cells into slots: copies inputs, rates, starting step, difference
// table, and queues the slot.  One workgroup per (slot, cell) pair.
__global__ void __launch_bounds__(kBlock) k_admit(Slots s, DeviceNet n, AdmitArgs a) {
    extern __shared__ double smem[];
    __shared__ SlotCtl cs;
    __shared__ double red[kWaves], phit[5];
    const int idx = blockIdx.x;
    if (idx >= a.count) return;
    const int slot = a.slots[idx];
    const long long cell = a.cells[idx];
    const int S = s.S;
    double *xs = smem;
    double *f0 = xs + S;
    double *rate = f0 + S;
    double *f1 = rate + n.R;
    double *phi = s.phi + size_t(slot) * 5;
    double *k = s.k + size_t(slot) * n.R;
    double *D = s.D + size_t(slot) * kDRows * S;
    if (threadIdx.x == 0) {
        phi[0] = a.T[cell]; phi[1] = a.nH[cell]; phi[2] = a.Av[cell]; phi[3] = a.zeta[cell]; phi[4] = a.G0[cell];
        SlotCtl z = {};
        z.t = 0.0;
        z.t_end = a.t_end[cell];
        z.rtol = a.rtol_c ? a.rtol_c[cell] : a.rtol;
        z.atol = a.atol_c ? a.atol_c[cell] : a.atol;
        z.newton_tol = a.newton_tol > 0.0 ? a.newton_tol
                                          : fmax(10.0 * kURound / z.rtol, fmin(0.03, sqrt(z.rtol)));
        z.q = s.method == ABDF_METHOD_ESDIRK5 ? 5 : 1;
        z.stage = 2;
        z.status = kRunning;
        z.j_fresh = 1;
        z.lu_valid = 0;
        z.cell = int32_t(cell);
        z.tc = a.tc ? a.tc[cell] : 0.0;
        cs = z;
    }
    bool bad = false;
    for (int i = threadIdx.x; i < S; i += kBlock) {
        const double v = a.x0[size_t(cell) * S + i];
        xs[i] = v;
        D[i] = v;
        for (int j = 1; j < kDRows; ++j) D[j * S + i] = 0.0;
        s.xJ[size_t(slot) * S + i] = v;
        bad |= !isfinite(v);
    }
    __syncthreads();
    const double T = phi[0], nH = phi[1], Av = phi[2], zeta = phi[3], G0 = phi[4];
    bad |= !(isfinite(T) && T > 0.0 && isfinite(nH) && nH > 0.0 && isfinite(Av) && isfinite(zeta) &&
             zeta >= 0.0 && isfinite(G0) && G0 >= 0.0 && isfinite(cs.t_end) && cs.t_end >= 0.0 &&
             isfinite(cs.rtol) && cs.rtol > 0.0 && isfinite(cs.atol) && cs.atol >= 0.0 && isfinite(cs.tc) &&
             cs.tc >= 0.0);
    bad = block_any(bad, red);
    if (bad) {
        finish_slot(s, slot, cs, ABDF_CELL_BAD_INPUT);
        __syncthreads();
        if (threadIdx.x == 0) s.ctl[slot] = cs;
        return;
    }
    if (s.tape_stop && s.tape_stop[cell] <= 0) {
        // a forward re-run that does not need this cell
        finish_slot(s, slot, cs, ABDF_CELL_OK);
        __syncthreads();
        if (threadIdx.x == 0) s.ctl[slot] = cs;
        return;
    }
    cell_rates(n, phi, k);
    __syncthreads();
    if (cs.t_end == 0.0) {
        finish_slot(s, slot, cs, ABDF_CELL_OK);
        __syncthreads();
        if (threadIdx.x == 0) s.ctl[slot] = cs;
        return;
    }
    // starting step (Hairer, Norsett & Wanner, Solving ODEs I, Sec. II.4), for
    // the method's order: 1 (BDF's first step) or 5 (ESDIRK)
    const bool rk = s.method == ABDF_METHOD_ESDIRK5;
    cell_rhs(n, k, xs, rate, f0);
    {
        // rates that overflow at the initial state leave no step to take
        bool nf = false;
        for (int i = threadIdx.x; i < S; i += kBlock) nf |= !isfinite(f0[i]);
        if (block_any(nf, red)) {
            if (threadIdx.x == 0) cs.n_rhs = 1;
            __syncthreads();
            finish_slot(s, slot, cs, ABDF_CELL_NONFINITE);
            __syncthreads();
            if (threadIdx.x == 0) s.ctl[slot] = cs;
            return;
        }
    }
    const double rtol = cs.rtol;
    double s0 = 0.0, s1 = 0.0;
    for (int i = threadIdx.x; i < S; i += kBlock) {
        const double sc = atol_of(s, cs, i) + rtol * fabs(xs[i]);
        s0 += (xs[i] / sc) * (xs[i] / sc);
        s1 += (f0[i] / sc) * (f0[i] / sc);
    }
    const double d0 = sqrt(block_sum(s0, red) / S);
    const double d1 = sqrt(block_sum(s1, red) / S);
    double h0 = (d0 < 1e-5 || d1 < 1e-5) ? 1e-6 : 0.01 * d0 / d1;
    h0 = fmin(h0, cs.t_end);
    // x1 = x0 + h0 f0 (kept in f1 as scratch, then f1 = f(x1))
    double *x1 = f1 + S;
    for (int i = threadIdx.x; i < S; i += kBlock) x1[i] = xs[i] + h0 * f0[i];
    if (s.tvar && cs.tc > 0.0) {
        // the trial evaluation at t = h0
        phi_at(s, slot, cs.tc, h0, phit);
        __syncthreads();
        cell_rates(n, phit, k);
    }
    __syncthreads();
    cell_rhs(n, k, x1, rate, f1);
    double s2 = 0.0;
    for (int i = threadIdx.x; i < S; i += kBlock) {
        const double sc = atol_of(s, cs, i) + rtol * fabs(xs[i]);
        const double v = (f1[i] - f0[i]) / sc;
        s2 += v * v;
    }
    const double d2 = sqrt(block_sum(s2, red) / S) / h0;
    const double mx = fmax(d1, d2);
    const double h1 = mx <= 1e-15 ? fmax(1e-6, h0 * 1e-3) : (rk ? pow(0.01 / mx, 1.0 / 6.0) : sqrt(0.01 / mx));
    double h = s.h0 > 0.0 ? fmin(s.h0, cs.t_end) : fmin(fmin(100.0 * h0, h1), cs.t_end);
    if (s.h_max > 0.0) h = fmin(h, s.h_max);
    for (int i = threadIdx.x; i < S; i += kBlock) D[S + i] = rk ? f0[i] : h * f0[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        cs.h = h;
        cs.n_rhs = 2;
        cs.n_jac = 1;
        s.ctl[slot] = cs;
    }
    queue_slot(s, slot);
}

// Threads of the standalone right-hand side's per-cell kernel: its LDS (the
// rates) allows two workgroups per CU, so each takes sixteen waves and the CU
// runs its full 32.
constexpr int kRhsThreads = 1024;

// Streaming right-hand side (k_rhs_stream): a
// workgroup of kRhsStreamThreads evaluates one cell after another, and each
// thread keeps for the whole launch its reactant pairs and its wave's lane
// groups of the species sums (two 16-bit entries a register), so the sums read
// LDS only and the next cell's inputs can be in flight while they run.  The
// lanes sum the entries of species_gather in the same order; the padding
// reads a -0.0 placed after the rates instead of being skipped (adding -0.0
// changes no sum, signed zeros included), so no entry needs a test, and a
// one-reactant rate takes a 1.0 placed after x as its second factor.
// LDS: rate [R], -0.0, x [S], 1.0, from the start of the dynamic block.  A
// resident entry is the rate's LDS address | nu in 3 bits, two's complement,
// so the sums read LDS at the entry's own address (the kernels have no static
// LDS, so the dynamic block starts at address 0 and every address fits 16
// bits).  Requires S <= kRhsStreamThreads, R < 8191, at most kGPW * 8 lane
// groups of at most kRhsResidentLen entries, and R <= kKU * kRhsStreamThreads
// (rhs_stream_shape checks).
constexpr int kRhsStreamThreads = 512;
template <int kKU, int kGPW>
struct RhsResident {
    static constexpr int NT = kRhsStreamThreads, NW = NT / 64, kE = kRhsResidentLen / 2;
    static constexpr int kB = kGPW * kKU >= 16 ? 4 : 8;   // LDS reads in flight per lane, as registers allow
    uint32_t ab[kKU];
    uint32_t ent[kGPW][kE];
    int red[kGPW], L[kGPW], steps[kGPW];

    // reactant pairs as LDS byte offsets into x (the 1.0 at x[S] for none)
    __device__ __forceinline__ void load_pairs(const DeviceNet &n) {
#pragma unroll
        for (int u = 0; u < kKU; ++u) {
            const int r = threadIdx.x + u * NT;
            const int w = r < n.R ? n.rx_ab[r] : 0;
            const int a = w & 0xffff, b = (w >> 16) & 0xffff;
            ab[u] = uint32_t(a * 8) | (uint32_t(b == 0xffff ? n.S : b) * 8u << 16);
        }
    }

    __device__ __forceinline__ void load(const DeviceNet &n, const double *smem) {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int R = n.R;
        load_pairs(n);
        // the LDS address of rate[0]
        const uint32_t lds0 = uint32_t(size_t((const __attribute__((address_space(3))) char *)smem));
        const uint32_t pad = (lds0 + uint32_t(R) * 8u) | 1u;   // +1 times the -0.0 after the rates
        auto conv = [lds0](int32_t w) { return (lds0 + uint32_t(w & ~7)) | (uint32_t((w & 7) - 4) & 7u); };
#pragma unroll
        for (int gi = 0; gi < kGPW; ++gi) {
            const int g = wave + gi * NW;
            const bool has = g < n.n_sgroup;
            const int mine = has ? n.sg_lane[g * 64 + lane] : 0;
            red[gi] = has ? n.sg_red[g * 64 + lane] : -1;
            const int lw = has ? __builtin_amdgcn_readfirstlane(n.sg_len[g]) : 0;
            L[gi] = lw & 0xffffff;
            steps[gi] = lw >> 24;
            if (L[gi] > 0) {
                // every load in flight at once: indexes past the group's
                // longest lane are clamped to its last row, their values unused
                const int32_t *e = n.sg_ent + n.sg_base[g] + lane;
                int32_t v[kRhsResidentLen];
#pragma unroll
                for (int j = 0; j < kRhsResidentLen; ++j) v[j] = e[min(j, L[gi] - 1) * 64];
#pragma unroll
                for (int j = 0; j < kE; ++j) {
                    const uint32_t lo = 2 * j < mine ? conv(v[2 * j]) : pad;
                    const uint32_t hi = 2 * j + 1 < mine ? conv(v[2 * j + 1]) : pad;
                    ent[gi][j] = lo | (hi << 16);
                }
            } else {
#pragma unroll
                for (int j = 0; j < kE; ++j) ent[gi][j] = pad | (pad << 16);
            }
        }
    }

    __device__ __forceinline__ static void init_lds(const DeviceNet &n, double *smem) {
        if (threadIdx.x == 0) {
            smem[n.R] = -0.0;
            smem[n.R + 1 + n.S] = 1.0;
        }
    }

    // rate[r] = k_r x_a x_b for this thread's reactions (x in LDS)
    __device__ __forceinline__ void rates(const DeviceNet &n, const double (&kr)[kKU], double *smem) const {
        const char *xb = reinterpret_cast<const char *>(smem + n.R + 1);
#pragma unroll
        for (int u = 0; u < kKU; ++u) {
            const int r = threadIdx.x + u * NT;
            const double xa = *reinterpret_cast<const double *>(xb + (ab[u] & 0xffffu));
            const double xc = *reinterpret_cast<const double *>(xb + (ab[u] >> 16));
            if (r < n.R) smem[r] = kr[u] * xa * xc;
        }
    }

    // out_i = sum_r nu_ir rate_r, written by each species' first lane
    __device__ __forceinline__ void sums(const DeviceNet &n, const double *smem, double *out) {
        // the entries are opaque to the compiler from one cell to the next,
        // so that it keeps them packed instead of hoisting what it derives from
        // them (offsets, coefficients) out of the cell loop into registers
#pragma unroll
        for (int gi = 0; gi < kGPW; ++gi)
#pragma unroll
            for (int j = 0; j < kE; ++j) asm volatile("" : "+v"(ent[gi][j]));
#pragma unroll
        for (int gi = 0; gi < kGPW; ++gi) {
            if (L[gi] == 0) continue;
            double acc = 0.0;
#pragma unroll
            for (int jb = 0; jb < kRhsResidentLen; jb += kB) {
                if (jb < L[gi]) {   // the same for the whole wave
                    double vv[kB], cf[kB];
#pragma unroll
                    for (int u = 0; u < kB; ++u) {
                        const int j = jb + u, sh = 16 * (j & 1);
                        const uint32_t w = ent[gi][j >> 1];
                        vv[u] = *(const __attribute__((address_space(3))) double *)size_t((w >> sh) & 0xfff8u);
                        cf[u] = double(int32_t(w << (29 - sh)) >> 29);
                    }
#pragma unroll
                    for (int u = 0; u < kB; ++u) acc += cf[u] * vv[u];
                }
            }
            const int q = red[gi] < 0 ? 0 : (red[gi] >> 7) & 127, m = red[gi] < 0 ? 1 : red[gi] & 127;
            for (int t = 0; t < steps[gi]; ++t) {
                const int off = 1 << t;
                const double o = __shfl_down(acc, off);
                if ((q & (2 * off - 1)) == 0 && q + off < m) acc += o;
            }
            if (red[gi] >= 0 && q == 0) out[red[gi] >> 14] = acc;
        }
    }
};

// Copies results of finished slots to the caller's arrays.
__global__ void __launch_bounds__(kBlock) k_harvest(Slots s, HarvestArgs h) {
    const int idx = blockIdx.x;
    if (idx == 0 && threadIdx.x == 0) s.q->nfin = 0;
    if (idx >= h.count) return;
    const int slot = h.slots[idx];
    const SlotCtl &c = s.ctl[slot];
    const long long cell = h.compact ? idx : c.cell;
    const int S = s.S;
    for (int i = threadIdx.x; i < S; i += kBlock) h.x_out[size_t(cell) * S + i] = s.D[size_t(slot) * kDRows * S + i];
    if (threadIdx.x == 0) {
        if (s.tape_len) s.tape_len[c.cell] = c.n_steps;
        h.status[cell] = c.status;
        if (h.stats) {
            abdf_cell_stats st;
            st.n_steps = c.n_steps;
            st.n_attempts = c.n_attempts;
            st.n_err_reject = c.n_err_reject;
            st.n_newton_fail = c.n_newton_fail;
            st.n_rhs = c.n_rhs;
            st.n_jac = c.n_jac;
            st.n_lu = c.n_lu;
            st.order = c.q;
            st.h = c.h;
            st.t = c.t;
            st.n_lu_fp64 = s.prec == ABDF_PREC_FP32_LU ? c.n_lu64 : c.n_lu;
            st.reserved = 0;
            h.stats[cell] = st;
        }
    }
}

// dk_r / dphi_j of one reaction for phi = (T, n_H, A_V, zeta, G0) (paper Sec. 2
// Kooij-Arrhenius and direct cosmic-ray laws, App. B.1 photo and cosmic-ray-
// induced photon laws), written without dividing by zeta or G0: the
// cosmic-ray and photo coefficients are linear in them.
__device__ __forceinline__ void rate_param_derivs(const DeviceNet &n, int r, const double *phi, double k,
                                                  double d[5]) {
    const double T = phi[0], nH = phi[1], Av = phi[2];
    const int t = n.rx_type[r];
    d[0] = d[1] = d[2] = d[3] = d[4] = 0.0;
    if (t == kTwoBody) {
        d[0] = k * (n.beta[r] + n.gamma[r] / T) / T;
        d[1] = k / nH;
    } else if (t == kCosmicRay) {
        d[3] = n.alpha[r];
    } else if (t == kCrPhoton) {
        d[0] = k * n.beta[r] / T;
        d[3] = n.alpha[r] * pow(T / 300.0, n.beta[r]) * (n.gamma[r] / (1.0 - n.albedo));
    } else {
        d[2] = -n.gamma[r] * k;
        d[4] = n.alpha[r] * exp(-n.gamma[r] * Av);
    }
}

// Copies the gradients of finished reverse slots to per-cell arrays: dL/dlog
// alpha_r = k_r dL/dk_r, dL/dx_0, and dL/dphi = sum_r dL/dk_r dk_r/dphi
// (per-thread sums in reaction order, then a fixed tree).
__global__ void __launch_bounds__(kBlock) k_adj_harvest(Slots s, DeviceNet n, AdjHarvestArgs h) {
    __shared__ double red[kWaves];
    const int idx = blockIdx.x;
    if (idx == 0 && threadIdx.x == 0) s.q->nfin = 0;
    if (idx >= h.count) return;
    const int slot = h.slots[idx];
    const int32_t fin = s.ctl[slot].status;
    if (fin == kWindowDone || fin == kSitsOut) return;   // the cell's result comes in a later pass
    const long long cell = s.ctl[slot].cell;
    const int S = s.S, R = s.R;
    const double *gk = s.g + size_t(slot) * R, *k = s.k + size_t(slot) * R, *phi = s.phi + size_t(slot) * 5;
    // a cell whose forward solve failed contributes zeros (its coefficients
    // may not even be finite, e.g. for a non-physical temperature)
    const bool ok = s.ctl[slot].status == ABDF_CELL_OK;
    if (h.g_cell)
        for (int r = threadIdx.x; r < R; r += kBlock) h.g_cell[size_t(cell) * R + r] = ok ? k[r] * gk[r] : 0.0;
    if (h.dx0)
        for (int i = threadIdx.x; i < S; i += kBlock) h.dx0[size_t(cell) * S + i] = s.x[size_t(slot) * S + i];
    if (h.dphi) {
        double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        for (int r = ok ? int(threadIdx.x) : R; r < R; r += kBlock) {
            double d[5];
            rate_param_derivs(n, r, phi, k[r], d);
            const double g = gk[r];
#pragma unroll
            for (int j = 0; j < 5; ++j) acc[j] += g * d[j];
        }
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const double v = block_sum(acc[j], red);
            if (threadIdx.x == 0) h.dphi[size_t(cell) * 5 + j] = v;
        }
    }
}

// out[r] = sum over cells of g_cell[c][r], cells in order.
__global__ void k_grad_sum(const double *g_cell, long long cells, int R, double *out) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    double acc = 0.0;
    for (long long c = 0; c < cells; ++c) acc += g_cell[size_t(c) * R + r];
    out[r] = acc;
}

// dL/dphi of one cell (one workgroup) from its dL/dlog alpha: five sums over
// reactions of g_r d log k_r / d phi_j (paper Sec. 2, App. B.1 rate laws).
__global__ void __launch_bounds__(kBlock) k_phys_grad(DeviceNet n, PhysArgs p, const double *g_cell, double *out) {
    __shared__ double red[kWaves];
    const long long c = blockIdx.x;
    const double T = p.T[c], nH = p.nH[c], zeta = p.zeta[c], G0 = p.G0[c];
    const double *g = g_cell + size_t(c) * n.R;
    double sT = 0.0, sN = 0.0, sA = 0.0, sZ = 0.0, sG = 0.0;
    for (int r = threadIdx.x; r < n.R; r += kBlock) {
        const int t = n.rx_type[r];
        const double gr = g[r];
        if (t == kTwoBody) {
            sT += gr * (n.beta[r] + n.gamma[r] / T) / T;
            sN += gr / nH;
        } else if (t == kCosmicRay) {
            sZ += gr / zeta;
        } else if (t == kCrPhoton) {
            sT += gr * n.beta[r] / T;
            sZ += gr / zeta;
        } else {
            sA += -n.gamma[r] * gr;
            sG += gr / G0;
        }
    }
    sT = block_sum(sT, red);
    sN = block_sum(sN, red);
    sA = block_sum(sA, red);
    sZ = block_sum(sZ, red);
    sG = block_sum(sG, red);
    if (threadIdx.x == 0) {
        double *o = out + size_t(c) * 5;
        o[0] = sT;
        o[1] = sN;
        o[2] = sA;
        o[3] = sZ;
        o[4] = sG;
    }
}

// ------------------------------------------------- component entry kernels --

__global__ void __launch_bounds__(kBlock) k_rates_only(DeviceNet n, PhysArgs p, double *k_out) {
    __shared__ double phi[5];
    const long long c = blockIdx.x;
    if (threadIdx.x == 0) {
        phi[0] = p.T[c]; phi[1] = p.nH[c]; phi[2] = p.Av[c]; phi[3] = p.zeta[c]; phi[4] = p.G0[c];
    }
    __syncthreads();
    cell_rates(n, phi, k_out + size_t(c) * n.R);
}

__global__ void __launch_bounds__(kRhsThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_rhs_only(DeviceNet n, const double *k, const double *x, double *f) {
    extern __shared__ double smem[];
    const long long c = blockIdx.x;
    double *xs = smem, *rate = xs + n.S;
    for (int i = threadIdx.x; i < n.S; i += kRhsThreads) xs[i] = x[size_t(c) * n.S + i];
    __syncthreads();
    cell_rhs<kRhsThreads, true>(n, k + size_t(c) * n.R, xs, rate, f + size_t(c) * n.S);
}

// The standalone right-hand side, streaming: each workgroup walks the cells
// blockIdx.x, blockIdx.x + gridDim.x, ...; the next cell's k and x are loaded
// into registers while the current cell's sums run (RhsResident).
template <int kKU, int kGPW>
__global__ void __launch_bounds__(kRhsStreamThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_rhs_stream(DeviceNet n, long long C, const double *__restrict__ k, const double *__restrict__ x,
             double *__restrict__ f) {
    using RR = RhsResident<kKU, kGPW>;
    constexpr int NT = kRhsStreamThreads;
    extern __shared__ double smem[];
    const int tid = threadIdx.x;
    const int S = n.S, R = n.R;
    RR rr;
    rr.load(n, smem);
    RR::init_lds(n, smem);
    double *xs = smem + R + 1;
    long long c = blockIdx.x;
    double kr[kKU], xr = 0.0;
    if (c < C) {
#pragma unroll
        for (int u = 0; u < kKU; ++u) kr[u] = tid + u * NT < R ? k[size_t(c) * R + tid + u * NT] : 0.0;
        if (tid < S) xr = x[size_t(c) * S + tid];
    }
    for (; c < C; c += gridDim.x) {
        const long long cn = c + gridDim.x;
        if (tid < S) xs[tid] = xr;
        __syncthreads();
        rr.rates(n, kr, smem);
        __syncthreads();
        if (cn < C) {
#pragma unroll
            for (int u = 0; u < kKU; ++u)
                if (tid + u * NT < R) kr[u] = k[size_t(cn) * R + tid + u * NT];
            if (tid < S) xr = x[size_t(cn) * S + tid];
        }
        rr.sums(n, smem, f + size_t(c) * S);
        __syncthreads();
    }
}

// Writes the unpadded S x S Newton matrix of each cell, kAsmRows rows a
// workgroup: the rows' Jacobian nonzeros (jacobian_values) go to LDS, and every
// entry is written as NewtonMatrixSource yields it to the factorisation's
// gather, a wave to a row, 64 columns at a time.  A call of 192 cells of 200
// species (61 MB written) took 194 us with one workgroup a cell, the nonzeros in
// global scratch allocated by the call and two integer divisions an entry, and
// takes 82 us.
constexpr int kAsmThreads = 256, kAsmRows = 16;   // rows: the blocks of jlong16

__global__ void __launch_bounds__(kAsmThreads) k_newton_matrix_only(DeviceNet n, const double *k, const double *x,
                                                                  const double *cvec, double *M) {
    extern __shared__ double smem[];
    const long long cell = blockIdx.y;
    const int S = n.S, r0 = blockIdx.x * kAsmRows, r1 = min(r0 + kAsmRows, S);
    double *xs = smem, *jv = xs + S;
    for (int i = threadIdx.x; i < S; i += kAsmThreads) xs[i] = x[size_t(cell) * S + i];
    const int e0 = n.jrow_ptr[r0], e1 = n.jrow_ptr[r1];
    __syncthreads();
    const int l0 = n.jlong16_ptr[blockIdx.x], l1 = n.jlong16_ptr[blockIdx.x + 1];
    jacobian_values<kAsmThreads>(n, k + size_t(cell) * n.R, xs, jv, e0, e1, n.jlong16 + l0, l1 - l0);
    __syncthreads();
    const double c = cvec[cell];
    const int lane = threadIdx.x & 63;
    for (int i = r0 + wave_of(threadIdx.x); i < r1; i += kAsmThreads / 64) {
        const NewtonMatrixSource<double> src{n.jmask, n.jbase, n.nbw, jv, c};
        double *row = M + (size_t(cell) * S + i) * S;
        for (int c0 = 0; c0 < S; c0 += 64) {
            const int j = c0 + lane;
            auto w = src.row(i, c0);
            w.base -= e0;
            if (j < S) row[j] = src.entry(w, i, j);
        }
    }
}

// The same for networks whose 16 densest rows do not fit in the LDS (more than
// some 1200 species): a workgroup to a row, every entry's terms from global memory.
__global__ void __launch_bounds__(kAsmThreads) k_newton_matrix_large(DeviceNet n, const double *k, const double *x,
                                                                   const double *cvec, double *M) {
    const int S = n.S, i = blockIdx.x;
    const size_t cell = blockIdx.y;
    const double *kc = k + cell * n.R, *xc = x + cell * S;
    const double c = cvec[cell];
    double *row = M + (cell * S + i) * S;
    for (int j = threadIdx.x; j < S; j += kAsmThreads) {
        const int e = n.jidx[size_t(i) * n.NP + j];
        double v = 0.0;
        for (int t = e < 0 ? 0 : n.jterm_ptr[e], t1 = e < 0 ? 0 : n.jterm_ptr[e + 1]; t < t1; ++t) {
            const int w = n.jt_rx_other[t], other = (w & 0xffff) - 1;
            double p = n.jt_coef[t] * kc[w >> 16];
            if (other >= 0) p *= xc[other];
            v += p;
        }
        row[j] = (i == j ? 1.0 : 0.0) - c * v;
    }
}

// Matrix-core lane-layout check: D = A B for integer-valued A (16x4), B (4x16).
__global__ void k_selftest(int *bad) {
    const int l = threadIdx.x;
    auto Aval = [](int i, int k) { return double((i * 7 + k * 3) % 11 - 5); };
    auto Bval = [](int k, int j) { return double((k * 5 + j * 2) % 13 - 6); };
    f64x4 cd = {0, 0, 0, 0};
    cd = Mfma<double>::mma(Aval(l & 15, l >> 4), Bval(l >> 4, l & 15), cd);
    f32x4 cf = {0, 0, 0, 0};
    cf = Mfma<float>::mma(float(Aval(l & 15, l >> 4)), float(Bval(l >> 4, l & 15)), cf);
    int nb = 0;
    for (int v = 0; v < 4; ++v) {
        const int j = l & 15;
        double ref_d = 0.0, ref_f = 0.0;
        const int id = Mfma<double>::row(l, v), jf = Mfma<float>::row(l, v);
        for (int k = 0; k < 4; ++k) {
            ref_d += Aval(id, k) * Bval(k, j);
            ref_f += Aval(jf, k) * Bval(k, j);
        }
        nb += (cd[v] != ref_d) + (double(cf[v]) != ref_f);
    }
    // wave arg-max: several value patterns with ties, checked against brute force
    for (int pat = 0; pat < 4; ++pat) {
        auto val = [pat](int i) {
            return pat == 0 ? double((i * 37) % 64) : pat == 1 ? double((i * 13) % 7) : pat == 2 ? 1.0 : double(i % 5 == 3 ? 9 : -1);
        };
        double v = val(l);
        int k = (l * 29 + pat) % 64;
        double bv = val(0);
        int bk = (pat) % 64;
        for (int i = 1; i < 64; ++i) {
            const double vi = val(i);
            const int ki = (i * 29 + pat) % 64;
            if (vi > bv || (vi == bv && ki < bk)) { bv = vi; bk = ki; }
        }
        double v2 = v;
        int k2 = k;
        wave_argmax(v, k);
        nb += (v != bv) + (k != bk);
        wave_argmax_ballot(v2, k2);
        nb += (v2 != bv) + (k2 != bk);
    }
    {
        double v = -1.0;     // no lane with a candidate
        int k = l;
        wave_argmax_ballot(v, k);
        nb += !(v < 0.0);
    }
    atomicAdd(bad, nb);
}

// v[0..n) = value (counters cleared by a kernel rather than a memset node)
__global__ void k_fill_i32(int32_t *v, int32_t value, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = value;
}

// ------------------------------------------------------------- launchers --

hipError_t launch_fill_i32(int32_t *v, int32_t value, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, st, v, value, n);
    return hipGetLastError();
}

// The streaming right-hand side's instantiation for a network: lanes groups
// per wave (1 or 2) and reactions per thread (ku), or false when the network
// does not fit them.
static bool rhs_stream_shape(const DeviceNet &n, int &ku, int &gpw) {
    constexpr int NW = kRhsStreamThreads / 64;
    if (n.S > kRhsStreamThreads || n.R >= 8191 || n.sg_maxlen > kRhsResidentLen || n.n_sgroup > 2 * NW) return false;
    gpw = n.n_sgroup <= NW ? 1 : 2;
    const int need = (n.R + kRhsStreamThreads - 1) / kRhsStreamThreads;
    ku = need <= 2 ? 2 : need <= 4 ? 4 : need <= 8 ? 8 : need <= 12 ? 12 : 16;
    return !(gpw == 2 && ku > 12);   // <16, 2> would spill
}

#define ABDF_RHS_STREAM_PICK(K)                                                                              \
    (gpw == 1 ? (ku == 2 ? (const void *)&K<2, 1> : ku == 4 ? (const void *)&K<4, 1> : ku == 8 ? (const void *)&K<8, 1> \
                 : ku == 12 ? (const void *)&K<12, 1> : (const void *)&K<16, 1>)                                         \
              : (ku == 2 ? (const void *)&K<2, 2> : ku == 4 ? (const void *)&K<4, 2> : ku == 8 ? (const void *)&K<8, 2> \
                 : (const void *)&K<12, 2>))

int lu_leading_dim(int NP) { return lu_ld(NP); }

size_t dinv_bytes(int NP, int prec) {
    return prec == ABDF_PREC_FP32_LU ? lu2_dinv_elems<float>(NP) * sizeof(float)
                                     : lu2_dinv_elems<double>(NP) * sizeof(double);
}

#define LAUNCH_CHECK() hipGetLastError()

hipError_t launch_admit(const Slots &s, const DeviceNet &n, const AdmitArgs &a, size_t lds, hipStream_t st) {
    if (a.count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_admit, dim3(a.count), dim3(kBlock), lds, st, s, n, a);
    return LAUNCH_CHECK();
}

hipError_t launch_harvest(const Slots &s, const HarvestArgs &h, hipStream_t st) {
    hipLaunchKernelGGL(k_harvest, dim3(h.count > 0 ? h.count : 1), dim3(kBlock), 0, st, s, h);
    return LAUNCH_CHECK();
}

hipError_t launch_adj_harvest(const Slots &s, const DeviceNet &n, const AdjHarvestArgs &h, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_harvest, dim3(h.count > 0 ? h.count : 1), dim3(kBlock), 0, st, s, n, h);
    return LAUNCH_CHECK();
}

hipError_t launch_grad_sum(const double *g_cell, long long cells, int R, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_grad_sum, dim3((R + 255) / 256), dim3(256), 0, st, g_cell, cells, R, out);
    return LAUNCH_CHECK();
}

hipError_t launch_phys_grad(const DeviceNet &n, const PhysArgs &p, long long cells, const double *g_cell,
                            double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_phys_grad, dim3(cells), dim3(kBlock), 0, st, n, p, g_cell, out);
    return LAUNCH_CHECK();
}

hipError_t launch_rates(const DeviceNet &n, const PhysArgs &p, long long cells, double *k, hipStream_t st) {
    hipLaunchKernelGGL(k_rates_only, dim3(cells), dim3(kBlock), 0, st, n, p, k);
    return LAUNCH_CHECK();
}

hipError_t plan_rhs(const DeviceNet &n, long long cells, RhsPlan &p) {
    int ku = 0, gpw = 0;
    p = RhsPlan{};
    if (rhs_stream_shape(n, ku, gpw)) {
        p.fn = ABDF_RHS_STREAM_PICK(k_rhs_stream);
        p.lds = sizeof(double) * (size_t(n.S) + n.R + 2);
        p.threads = kRhsStreamThreads;
        int dev = 0, ncu = 0, nb = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, p.fn, kRhsStreamThreads, p.lds);
        if (e != hipSuccess) return e;
        p.grid = std::min<long long>(cells, std::max(1LL, (long long)nb * ncu));
        return hipSuccess;
    }
    p.fn = reinterpret_cast<const void *>(&k_rhs_only);
    p.lds = sizeof(double) * (size_t(n.S) + n.R);
    p.threads = kRhsThreads;
    p.grid = cells;
    return hipSuccess;
}

hipError_t launch_rhs_planned(const RhsPlan &p, const DeviceNet &n, long long cells, const double *k, const double *x,
                              double *f, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
    DeviceNet nn = n;
    long long C = cells;
    const double *kk = k, *xx = x;
    double *ff = f;
    void *args_only[] = {&nn, &kk, &xx, &ff};
    void *args_stream[] = {&nn, &C, &kk, &xx, &ff};
    void **args = p.fn == reinterpret_cast<const void *>(&k_rhs_only) ? args_only : args_stream;
    return hipExtLaunchKernel(p.fn, dim3(unsigned(p.grid)), dim3(p.threads), args, p.lds, st, start, stop, 0);
}

hipError_t launch_newton_matrix(const DeviceNet &n, long long cells, const double *k, const double *x,
                                const double *c, double *M, hipStream_t st) {
    // grid.y holds at most 65535 cells
    const size_t lds = sizeof(double) * (size_t(n.S) + size_t(std::max(n.asm_nnz, 1)));
    const bool large = lds > kMaxLds;
    const auto kernel = large ? k_newton_matrix_large : k_newton_matrix_only;
    const unsigned blocks = large ? unsigned(n.S) : unsigned((n.S + kAsmRows - 1) / kAsmRows);
    for (long long c0 = 0; c0 < cells; c0 += 65535) {
        const unsigned m = unsigned(std::min<long long>(65535, cells - c0));
        hipLaunchKernelGGL(kernel, dim3(blocks, m), dim3(kAsmThreads), large ? 0 : lds, st, n,
                           k + size_t(c0) * n.R, x + size_t(c0) * n.S, c + c0, M + size_t(c0) * n.S * n.S);
        const hipError_t e = LAUNCH_CHECK();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_selftest(int *bad, hipStream_t st) {
    hipLaunchKernelGGL(k_selftest, dim3(1), dim3(64), 0, st, bad);
    return LAUNCH_CHECK();
}

}  // namespace abdf
