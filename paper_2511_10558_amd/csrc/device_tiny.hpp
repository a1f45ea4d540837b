// Step attempts of cells with at most 64 species: one wave per cell, a lane per
// species, and everything an attempt touches in LDS and registers: the rate
// coefficients, the network's reaction and species-sum tables, the Jacobian
// (dense) and the inverses of the Newton matrix's triangular factors.
//
// At this size an attempt is a chain of latencies, not of work (12 species:
// 2 kB of factors), so what counts is that no step of the chain leaves the
// compute unit or waits for another wave.  The arithmetic and the order of every
// sum are those of the wide kernel.
#pragma once

#include "device_step.hpp"

namespace abdf {

// LDS layout of a network's tiny-cell kernel (offsets in bytes): the
// factorisation's own block (in T, or in T and FP64 in turn), then the rest.
template <typename T, bool kFp64Too>
struct TinyLayout {
    int S, R, NP, ld, ng, nent;
    size_t J, k, rate, xs, f, ab, ent, lane, red, len, base, total;
    __host__ __device__ TinyLayout(const DeviceNet &n) {
        S = n.S;
        R = n.R;
        NP = n.NP;
        ng = n.n_sgroup;
        nent = n.sg_total;
        ld = S | 1;   // odd: a column's rows lie in different banks
        size_t o = lu2_lds_bytes<T, 1>(NP);
        if (kFp64Too && lu2_lds_bytes<double, 1>(NP) > o) o = lu2_lds_bytes<double, 1>(NP);
        o = (o + 15) / 16 * 16;
        auto part = [&o](size_t bytes) {
            const size_t at = o;
            o += (bytes + 7) / 8 * 8;
            return at;
        };
        J = part(size_t(S) * ld * 8);
        k = part(size_t(R) * 8);
        rate = part(size_t(R) * 8);
        xs = part(64 * 8);
        f = part(64 * 8);
        ab = part(size_t(R) * 4);
        ent = part(size_t(nent) * 4);
        lane = part(size_t(ng) * 64 * 4);
        red = part(size_t(ng) * 64 * 4);
        len = part(size_t(ng) * 4);
        base = part(size_t(ng) * 4);
        total = o;
    }
};

// The entries of M = I - c J from the dense J in LDS; the identity's beyond S.
template <typename T>
struct TinySource {
    const double *J;
    int S, ld;
    double c;
    struct Row { int32_t i; };
    __device__ __forceinline__ Row row(int r, int) const { return {r}; }
    __device__ __forceinline__ T entry(const Row &, int i, int j) const {
        const bool in = i < S && j < S;
        const double v = J[in ? i * ld + j : 0];
        return T((i == j ? 1.0 : 0.0) - c * (in ? v : 0.0));
    }
};

// kFp64Too (T = float): the cell's factors may also be FP64.  What concerns the
// factors is a template of their type U.
template <typename T, int kTiles, bool kFp64Too>
struct TinyCell {
    int S, R, NP, ld, ng;
    unsigned char *lu;       // lu_factor_left's LDS block
    double *J, *k, *rate, *xs, *f;
    int32_t *ab, *ent, *lane, *red, *len, *base;

    __device__ __forceinline__ TinyCell(const DeviceNet &n, unsigned char *smem) {
        const TinyLayout<T, kFp64Too> l(n);
        S = l.S;
        R = l.R;
        NP = l.NP;
        ld = l.ld;
        ng = l.ng;
        lu = smem;
        J = reinterpret_cast<double *>(smem + l.J);
        k = reinterpret_cast<double *>(smem + l.k);
        rate = reinterpret_cast<double *>(smem + l.rate);
        xs = reinterpret_cast<double *>(smem + l.xs);
        f = reinterpret_cast<double *>(smem + l.f);
        ab = reinterpret_cast<int32_t *>(smem + l.ab);
        ent = reinterpret_cast<int32_t *>(smem + l.ent);
        lane = reinterpret_cast<int32_t *>(smem + l.lane);
        red = reinterpret_cast<int32_t *>(smem + l.red);
        len = reinterpret_cast<int32_t *>(smem + l.len);
        base = reinterpret_cast<int32_t *>(smem + l.base);
        const int t = threadIdx.x;
        for (int r = t; r < R; r += 64) ab[r] = n.rx_ab[r];
        for (int e = t; e < l.nent; e += 64) ent[e] = n.sg_ent[e];
        for (int e = t; e < ng * 64; e += 64) {
            lane[e] = n.sg_lane[e];
            red[e] = n.sg_red[e];
        }
        for (int g = t; g < ng; g += 64) {
            len[g] = n.sg_len[g];
            base[g] = n.sg_base[g];
        }
    }

    __device__ __forceinline__ void load_rates(const double *kg) {
        for (int r = threadIdx.x; r < R; r += 64) k[r] = kg[r];
        wave_lds_order();
    }

    // f_i of this lane's species (0 past the last): rates, then the species
    // sums in the layout and order of species_gather.
    __device__ __forceinline__ double rhs(double x) {
        const int t = threadIdx.x;
        if (t < S) xs[t] = x;
        wave_lds_order();
        for (int r = t; r < R; r += 64) {
            const int w = ab[r], a = w & 0xffff, b = (w >> 16) & 0xffff;
            double v = k[r] * xs[a];
            if (b != 0xffff) v *= xs[b];
            rate[r] = v;
        }
        wave_lds_order();
        return sums();
    }

    // sum_r nu_ir rate_r of this lane's species
    __device__ __forceinline__ double sums() {
        const int t = threadIdx.x;
        for (int g = 0; g < ng; ++g) {
            const int mine = lane[g * 64 + t], rd = red[g * 64 + t];
            const int lw = __builtin_amdgcn_readfirstlane(len[g]);
            const int L = lw & 0xffffff, steps = lw >> 24;
            const int32_t *e = ent + __builtin_amdgcn_readfirstlane(base[g]) + t;
            double acc = 0.0;
            for (int jb = 0; jb < L; jb += 4) {
                int w[4];
                double vv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = jb + u < mine ? e[(jb + u) * 64] : 4;   // 4: coefficient 0, entry 0
#pragma unroll
                for (int u = 0; u < 4; ++u) vv[u] = rate[w[u] >> 3];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (jb + u < mine) acc += double((w[u] & 7) - 4) * vv[u];
            }
            const int q = rd < 0 ? 0 : (rd >> 7) & 127, m = rd < 0 ? 1 : rd & 127;
            for (int st = 0; st < steps; ++st) {
                const int off = 1 << st;
                const double o = __shfl_down(acc, off);
                if ((q & (2 * off - 1)) == 0 && q + off < m) acc += o;
            }
            if (rd >= 0 && q == 0) f[rd >> 14] = acc;
        }
        wave_lds_order();
        return t < S ? f[t] : 0.0;
    }

    // J(x_J), dense, by way of its nonzeros (jv: nnzJ doubles of the slot)
    __device__ __forceinline__ void jacobian(const DeviceNet &n, const double *xJ, double *jv) {
        if (int(threadIdx.x) < S) xs[threadIdx.x] = xJ[threadIdx.x];
        wave_lds_order();
        jacobian_values<64, 2, 4>(n, k, xs, jv);
        // a lane scatters what another one wrote (jacobian_values takes the long
        // lists in an order of their own)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        scatter(n, jv);
    }
    // the nonzeros (global memory) into the dense J
    __device__ __forceinline__ void scatter(const DeviceNet &n, const double *jv) {
        for (int e = threadIdx.x; e < S * ld; e += 64) J[e] = 0.0;
        wave_lds_order();
        for (int e = threadIdx.x; e < n.nnzJ; e += 64) J[n.jrow[e] * ld + n.jcol[e]] = jv[e];
        wave_lds_order();
    }

    // M = I - c J factored; the inverses of its triangles and the row order stay
    // in LDS for the solves.
    template <typename U>
    __device__ __forceinline__ void factor(const Slots &s, int slot, double c) {
        lu_factor_left<U, 1, kTiles>(SlotStorage<U>{slot_lu<U>(s, slot), s.lda}, NP, s.perm + size_t(slot) * NP,
                                     slot_dinv<U>(s, slot), nullptr, lu, TinySource<U>{J, S, ld, c});
        wave_lds_order();
    }

    // y = D b for a triangle's inverse D in LDS (D: inv(L) if lower, else
    // inv(U)): 16 lanes to a row, with the products and the order of
    // lu_solve_left's diagonal blocks.  b, y in LDS.  A lane group reads the
    // entries of P rows (all of them up to 32 species) before it uses any: rows
    // two at a time, a solve of 12 species took 2.5 us, and takes 1.9.
    template <typename U>
    __device__ __forceinline__ void triangle(const U *D, bool lower, const double *b, double *y) const {
        constexpr int VW = 16 / int(sizeof(U)), H = (16 * kTiles + 16 * VW - 1) / (16 * VW);
        constexpr int P = kTiles == 2 ? 8 : 4;
        const int N = min(NP, S + (S & 1));
        const int lane16 = threadIdx.x & 15, row4 = threadIdx.x >> 4;
        double tv[H][VW];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int q = 0; q < VW; ++q) {
                const int c = VW * lane16 + 16 * VW * h + q;
                tv[h][q] = c < N ? b[c] : 0.0;
            }
        for (int r0 = 0; r0 < N; r0 += 4 * P) {
            U a[P][H][VW];
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int q = 0; q < VW; ++q) {
                        const int rr = min(r0 + 4 * p + row4, N - 1), c = VW * lane16 + 16 * VW * h + q;
                        const bool use = c < N && (lower ? c <= rr : c >= rr);
                        a[p][h][q] = D[rr * kLdb + (use ? c : rr)];
                    }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int r = r0 + 4 * p + row4, rr = min(r, N - 1);
                double acc = 0.0;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int c = VW * lane16 + 16 * VW * h;
                    double term[VW];
#pragma unroll
                    for (int q = 0; q < VW; ++q) {
                        const bool use = c + q < N && (lower ? c + q <= rr : c + q >= rr);
                        term[q] = use ? double(a[p][h][q]) * tv[h][q] : 0.0;
                    }
                    if constexpr (VW == 2)
                        acc += c < N ? term[0] + term[1] : 0.0;
                    else
                        acc += c < N ? (term[0] + term[1]) + (term[2] + term[3]) : 0.0;
                }
                acc = row_sum(acc);
                if (lane16 == 0 && r < N) y[r] = acc;
            }
        }
        wave_lds_order();
    }

    // This lane's entry of M^{-1} b, b given by lane.
    template <typename U>
    __device__ __forceinline__ double solve(double b) {
        const int t = threadIdx.x;
        const LuLds<U, 1> l(NP, lu);
        f[t] = t < S ? b : 0.0;
        wave_lds_order();
        xs[t] = t < NP ? f[l.perm[t]] : 0.0;
        wave_lds_order();
        triangle<U>(l.Xb, true, xs, f);
        triangle<U>(l.Ub, false, f, xs);
        return t < S ? xs[t] : 0.0;
    }

    // J(x_J) v, this lane's entry, reaction by reaction (cell_jvp)
    __device__ __forceinline__ double jvp(const double *xJ, double v) {
        const int t = threadIdx.x;
        if (t < S) {
            xs[t] = xJ[t];
            f[t] = v;
        }
        wave_lds_order();
        for (int r = t; r < R; r += 64) {
            const int w = ab[r], a = w & 0xffff, b = (w >> 16) & 0xffff;
            rate[r] = b == 0xffff ? k[r] * f[a] : k[r] * (f[a] * xs[b] + xs[a] * f[b]);
        }
        wave_lds_order();
        return sums();
    }

    // An interrupted cell's factors: the factorisation left its inverses and row
    // order in the slot's storage.
    template <typename U>
    __device__ __forceinline__ void restore(const Slots &s, int slot) {
        const U *di = slot_dinv<U>(s, slot);
        const LuLds<U, 1> l(NP, lu);
        for (int e = threadIdx.x; e < 64 * NP; e += 64) {
            l.Xb[(e >> 6) * kLdb + (e & 63)] = di[e];
            l.Ub[(e >> 6) * kLdb + (e & 63)] = di[kLuW * kLuW + e];
        }
        if (int(threadIdx.x) < NP) l.perm[threadIdx.x] = s.perm[size_t(slot) * NP + threadIdx.x];
        wave_lds_order();
    }
};

// The corrector of one attempt (newton_slot for a tiny cell).
template <typename T, int kTiles, bool kFp64Too>
__device__ __forceinline__ int newton_tiny(const Slots &s, int slot, StepLds<1> &L, SpeciesState &y,
                                           TinyCell<T, kTiles, kFp64Too> &cell, unsigned long long *t_rhs) {
    const int S = s.S, i = threadIdx.x;
    const bool own = i < S;
    SlotCtl &cs = L.cs;
    const double c = cs.c, c_lu = cs.c_lu, tol = cs.newton_tol;
    const bool refine = sizeof(T) == sizeof(float) && cs.lu_mode == kLuRefined32;
    const bool fp64 = kFp64Too && cs.lu_mode == kLu64;
    double eta_old = 0.0;
    int phase = kIter, m = 0;
    while (phase == kIter) {
        ++m;
        const unsigned long long t0 = t_rhs && i == 0 ? wall_clock64() : 0ull;
        const double f = cell.rhs(y.x);
        const double r = own ? c * f - y.psi - y.d : 0.0;
        if (t_rhs && i == 0) *t_rhs += wall_clock64() - t0;
        if (__ballot(own && !isfinite(f)) != 0) {
            phase = kFailed;
            break;
        }
        double delta = fp64 ? cell.template solve<double>(r) : cell.template solve<T>(r);
        if (refine) {
            const double jd = cell.jvp(s.xJ + size_t(slot) * S, delta);
            delta = delta + cell.template solve<T>(own ? r - (delta - c_lu * jd) : 0.0);
        }
        if (c != c_lu) delta = delta * (2.0 / (1.0 + c / c_lu));
        const double eta = sqrt(wg_square<1>(delta / y.scl, S, nullptr, L.red) / S);
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

}  // namespace abdf
