// Rate coefficients, right-hand side and Newton-matrix rows for one cell,
// evaluated cooperatively by one workgroup.
#pragma once

#include "device_common.hpp"
#include "network.hpp"

namespace abdf {

// k_r for one cell (paper Sec. 2 Kooij-Arrhenius and direct cosmic-ray forms,
// App. B.1 photo form and the cosmic-ray-induced photon form
// alpha (T/300)^beta E zeta / (1 - omega), E the reaction's efficiency kept in
// its gamma field, omega the network's dust albedo); two-body coefficients carry the factor n_H of the
// fractional-abundance state.  Written to global memory, coalesced over r.
template <int NT = kBlock>
__device__ inline void cell_rates(const DeviceNet &n, const double *phi, double *k) {
    const double T = phi[0], nH = phi[1], Av = phi[2], zeta = phi[3], G0 = phi[4];
    const double T300 = T / 300.0;
    // one exponential for the laws that have one, whatever the mix of laws
    // among a wave's reactions
    for (int r = thread_id(); r < n.R; r += NT) {
        const int t = n.rx_type[r];
        const double a = n.alpha[r], ga = n.gamma[r];
        const double e = exp(t == kTwoBody ? -ga / T : (t == kPhoto ? -ga * Av : 0.0));
        const double p = t == kTwoBody || t == kCrPhoton ? pow(T300, n.beta[r]) : 1.0;
        double v;
        if (t == kTwoBody) v = a * p * e * nH;
        else if (t == kCosmicRay) v = a * zeta;
        else if (t == kCrPhoton) v = a * p * (ga / (1.0 - n.albedo)) * zeta;
        else v = a * G0 * e;
        k[r] = v;
    }
}

// out_i = sum_r nu_ir v_r for per-reaction values v (LDS), in the wave layout
// of DeviceNet::sg_ent: each wave takes groups of 64 lanes; a lane sums its
// entries in order from zero, then the lanes of each species are added
// pairwise within the wave and the species' first lane writes out_i.
// Deterministic: the order of every sum is fixed by the layout, whichever
// wave takes a group.  The entries are loaded eight at a time before any is
// used, so the loads are in flight together.  Ends with a barrier.
template <int NT = kBlock>
__device__ __forceinline__ void species_gather(const DeviceNet &n, const double *v, double *out) {
    constexpr int kB = 8;
    const int tid = thread_id(), lane = tid & 63;
    for (int g = wave_of(tid); g < n.n_sgroup; g += NT / 64) {
        const int mine = n.sg_lane[g * 64 + lane];
        const int lw = n.sg_len[g];
        const int L = lw & 0xffffff, steps = lw >> 24;
        const int32_t *ent = n.sg_ent + n.sg_base[g] + lane;
        double acc = 0.0;
        for (int jb = 0; jb < L; jb += kB) {
            int w[kB];
#pragma unroll
            for (int u = 0; u < kB; ++u) w[u] = jb + u < mine ? ent[(jb + u) * 64] : 4;   // 4: coefficient 0, entry 0
            double vv[kB];
#pragma unroll
            for (int u = 0; u < kB; ++u) vv[u] = v[w[u] >> 3];
#pragma unroll
            for (int u = 0; u < kB; ++u)
                if (jb + u < mine) acc += double((w[u] & 7) - 4) * vv[u];
        }
        // the species' lanes pairwise; steps is the same for the whole wave
        const int red = n.sg_red[g * 64 + lane];
        const int q = red < 0 ? 0 : (red >> 7) & 127, m = red < 0 ? 1 : red & 127;
        for (int t = 0; t < steps; ++t) {
            const int off = 1 << t;
            const double o = __shfl_down(acc, off);
            if ((q & (2 * off - 1)) == 0 && q + off < m) acc += o;
        }
        if (red >= 0 && q == 0) out[red >> 14] = acc;
    }
    __syncthreads();
}

// f = nu . rate(x) for one cell.  x in LDS; k in global memory (one coalesced
// pass); rate[R] is LDS scratch; f may be LDS or global.
// Deterministic: every sum runs in a fixed order.
// kWide: more loads in flight per thread, for kernels with registers to spare.
template <int NT = kBlock, bool kWide = false>
__device__ __forceinline__ void cell_rhs(const DeviceNet &n, const double *__restrict__ k, const double *x,
                                double *rate, double *f) {
    // kU reactions per thread per pass, their loads issued before any use
    constexpr int kU = kWide ? 6 : 4;
    for (int r0 = thread_id(); r0 < n.R; r0 += kU * NT) {
        int ab[kU];
        double kr[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = r0 + u * NT;
            ab[u] = r < n.R ? n.rx_ab[r] : 0;
            kr[u] = r < n.R ? k[r] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = r0 + u * NT;
            const int a = ab[u] & 0xffff, b = (ab[u] >> 16) & 0xffff;
            double v = kr[u] * x[a];
            if (b != 0xffff) v *= x[b];
            if (r < n.R) rate[r] = v;
        }
    }
    __syncthreads();
    species_gather<NT>(n, rate, f);
}

// cell_rhs for a workgroup alone on its compute unit: the same values, with what
// the species sums need from memory asked for ahead.  A group's sums are its
// header, then its entries, then the rates they point to; the headers of a wave's
// first two groups and all entries of the first are on their way while the
// rates are formed, and each batch of entries used makes room for the same
// batch of the next group.  (A residual of 500 species 11.0 us a cell before, 8.9
// now with 96 cells in the FP32-LU form; 13.8 and 11.7 with 256 in FP64, where
// the solves beside it draw all the memory gives; of 200 species 5.3 and 5.0.)
template <int NT>
__device__ __forceinline__ void cell_rhs_ahead(const DeviceNet &n, const double *__restrict__ k, const double *x,
                                               double *rate, double *f) {
    constexpr int kU = 6, kB = 8, kM = kRhsResidentLen / kB, NW = NT / 64;
    static_assert(kRhsResidentLen % kB == 0 && kRhsSegment <= kRhsResidentLen, "a lane's entries in whole batches");
    const int tid = thread_id(), lane = tid & 63;
    struct Head { int mine, red, lw, base; };
    auto header = [&](int g) __attribute__((always_inline)) {
        const int gc = min(g, n.n_sgroup - 1);   // a network has at least one species, so one group
        Head h{n.sg_lane[gc * 64 + lane], n.sg_red[gc * 64 + lane], n.sg_len[gc], n.sg_base[gc]};
        return h;
    };
    int w[kM][kB];
    // entries past the group's longest lane are its last row's again, and not used
    auto entries = [&](const Head &h, int b) __attribute__((always_inline)) {
        const int L = h.lw & 0xffffff;
        if (b * kB < L) {
            const int32_t *e = n.sg_ent + h.base + lane;
#pragma unroll
            for (int u = 0; u < kB; ++u) w[b][u] = e[min(b * kB + u, L - 1) * 64];
        }
    };
    int g = wave_of(tid);
    Head h = header(g), hn = header(g + NW);
    for (int first = 0; first < n.R; first += kU * NT) {   // whole waves: every lane has entries to load
        const int r0 = first + tid;
        int ab[kU];
        double kr[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = min(r0 + u * NT, n.R - 1);
            ab[u] = n.rx_ab[r];
            kr[u] = k[r];
        }
        if (first == 0) {
#pragma unroll
            for (int b = 0; b < kM; ++b) entries(h, b);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = r0 + u * NT;
            const int p = ab[u] & 0xffff, q = (ab[u] >> 16) & 0xffff;
            double v = kr[u] * x[p];
            if (q != 0xffff) v *= x[q];
            if (r < n.R) rate[r] = v;
        }
    }
    __syncthreads();
    for (; g < n.n_sgroup; g += NW) {
        const Head hnn = header(g + 2 * NW);
        const int L = h.lw & 0xffffff, steps = h.lw >> 24;
        double acc = 0.0;
#pragma unroll
        for (int b = 0; b < kM; ++b) {
            if (b * kB < L) {
                double vv[kB];
#pragma unroll
                for (int u = 0; u < kB; ++u) vv[u] = rate[w[b][u] >> 3];
#pragma unroll
                for (int u = 0; u < kB; ++u)
                    if (b * kB + u < h.mine) acc += double((w[b][u] & 7) - 4) * vv[u];
            }
            if (g + NW < n.n_sgroup) entries(hn, b);
        }
        // a species of more than 64 lanes' entries (the lanes are then longer)
        for (int j = kM * kB; j < L; ++j) {
            const int wj = n.sg_ent[h.base + min(j, L - 1) * 64 + lane];
            if (j < h.mine) acc += double((wj & 7) - 4) * rate[wj >> 3];
        }
        const int q = h.red < 0 ? 0 : (h.red >> 7) & 127, m = h.red < 0 ? 1 : h.red & 127;
        for (int t = 0; t < steps; ++t) {
            const int off = 1 << t;
            const double o = __shfl_down(acc, off);
            if ((q & (2 * off - 1)) == 0 && q + off < m) acc += o;
        }
        if (h.red >= 0 && q == 0) f[h.red >> 14] = acc;
        h = hn;
        hn = hnn;
    }
    __syncthreads();
}

// J(x) y = nu . (d rate / dx) y for one cell: per reaction
// k_r (y_a x_b + x_a y_b) (k_r y_a for one reactant; the same expression gives
// 2 k_r x_a y_a for A + A), then the species sums of cell_rhs.  x, y in LDS;
// drate[R] LDS scratch.
template <int NT>
__device__ __forceinline__ void cell_jvp(const DeviceNet &n, const double *__restrict__ k, const double *x,
                                         const double *y, double *drate, double *out) {
    for (int r0 = thread_id(); r0 < n.R; r0 += 4 * NT) {
        int ab[4];
        double kr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u * NT;
            ab[u] = r < n.R ? n.rx_ab[r] : 0;
            kr[u] = r < n.R ? k[r] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u * NT;
            const int a = ab[u] & 0xffff, b = (ab[u] >> 16) & 0xffff;
            const double v = b == 0xffff ? kr[u] * y[a] : kr[u] * (y[a] * x[b] + x[a] * y[b]);
            if (r < n.R) drate[r] = v;
        }
    }
    __syncthreads();
    species_gather<NT>(n, drate, out);
}

// The Jacobian nonzeros J_e(x), first <= e < last, of one cell into jv[e - first]:
// each nonzero's terms summed in the order of its term list.  lists: the n_long of
// them that have more than kJacShort terms, longest first.  x in LDS; k in LDS or
// global memory.  Cooperative.
//
// A nonzero has 1.8 terms on average, but up to 52, and is a chain of three
// loads (its list's bounds, the terms, their coefficients).  The short lists
// come first, in the nonzeros' order: a thread works on kU of them at once, all
// their terms in flight together.  The long ones follow in the order of their
// lengths, so that the lanes of a wave finish together.  (In one pass every
// wave met a long list among its lanes and waited out its rounds of loads: a
// factorisation of 131 species with its Jacobian took 173 us, now 156; of 500
// 1105, now 1055; the FP32 one 713, now 658.)
template <int NT, int kU = 4, int kL = 8>
__device__ __forceinline__ void jacobian_values(const DeviceNet &n, const double *__restrict__ k, const double *x,
                                                double *jv, int first, int last, const int32_t *lists, int n_long) {
    constexpr int kT = kJacShort;
    auto term = [&](int w, double cf) {
        const int other = (w & 0xffff) - 1;
        double v = cf * k[w >> 16];
        if (other >= 0) v *= x[other];
        return v;
    };
    for (int e0 = first + thread_id(); e0 < last; e0 += kU * NT) {
        int t0[kU], t1[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = min(e0 + u * NT, last - 1);
            t0[u] = n.jterm_ptr[e];
            t1[u] = n.jterm_ptr[e + 1];
        }
        int w[kU][kT];
        double cf[kU][kT];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                const int at = min(t0[u] + t, t1[u] - 1);   // a nonzero has at least one term
                w[u][t] = n.jt_rx_other[at];
                cf[u][t] = n.jt_coef[at];
            }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            double v = 0.0;
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                const double p = term(w[u][t], cf[u][t]);
                if (t0[u] + t < t1[u]) v += p;
            }
            if (e0 + u * NT < last && t1[u] - t0[u] <= kT) jv[e0 + u * NT - first] = v;
        }
    }
    for (int i = thread_id(); i < n_long; i += NT) {
        const int e = lists[i], t1 = n.jterm_ptr[e + 1];
        double v = 0.0;
        for (int tb = n.jterm_ptr[e]; tb < t1; tb += kL) {
            int w[kL];
            double cf[kL];
#pragma unroll
            for (int t = 0; t < kL; ++t) {
                const int at = min(tb + t, t1 - 1);
                w[t] = n.jt_rx_other[at];
                cf[t] = n.jt_coef[at];
            }
#pragma unroll
            for (int t = 0; t < kL; ++t) {
                const double p = term(w[t], cf[t]);
                if (tb + t < t1) v += p;
            }
        }
        jv[e - first] = v;
    }
}

template <int NT, int kU = 4, int kL = 8>
__device__ __forceinline__ void jacobian_values(const DeviceNet &n, const double *__restrict__ k, const double *x,
                                                double *jv) {
    jacobian_values<NT, kU, kL>(n, k, x, jv, 0, n.nnzJ, n.jlong, n.n_jlong);
}

// Entries of M = I - c J of one cell where the factorisation gathers them:
// the 64-column words of the Jacobian's pattern give the nonzero of (i, j)
// (one word and one base per row and block column, shared by the lanes of a
// row); rows and columns beyond S are the identity's.
template <typename T>
struct NewtonMatrixSource {
    const uint64_t *jmask;   // [NP][nbw] pattern words
    const int32_t *jbase;    // [NP][nbw] index of the first nonzero of each word
    int nbw;
    const double *jv;        // the entries' values
    double c;
    // Entries are read in two passes, every row's word first and then every
    // value, so that no load waits behind a condition on an earlier one;
    // structural zeros load nothing.
    struct Row { uint64_t m; int32_t base; };
    __device__ __forceinline__ Row row(int i, int c0) const {
        const size_t w = size_t(i) * nbw + (c0 >> 6);
        return {jmask[w], jbase[w]};
    }
    __device__ __forceinline__ T entry(const Row &w, int i, int j) const {
        const int bit = j & 63;
        const bool nz = (w.m >> bit) & 1ull;
        const double jvv = nz ? jv[w.base + __popcll(w.m & ((1ull << bit) - 1ull))] : 0.0;
        return T((i == j ? 1.0 : 0.0) - c * jvv);
    }
};

}  // namespace abdf
