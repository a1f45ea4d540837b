// Factorisation and solve of a batch of the caller's own n x n FP64 matrices
// (n <= 512), one workgroup per matrix, in place: no padded copy is made and
// none is copied back.  (With the matrices copied to padded storage, factored
// there and copied back, a call of 256 matrices of order 500 moved another
// 2 GB and allocated 0.65 GB: 2.36 ms where the diagonal pivots hold, 1.37 ms
// now.)
#include "device_lu2.hpp"
#include "../../include/astrobdf.h"
#include "kernels.hpp"

#include <algorithm>

namespace abdf {

// ---------------------------------------------------------- factorisation --

// Waves of a factorisation, each holding four row tiles of the block column in
// its 256 VGPRs.
constexpr int kLuWaves = 8;

// Row i of the factors from storage row perm[i] to row i, 32 columns at a time:
// every row of the strip is read before any is written.  Rows that are in place
// (on the Newton matrices nearly all are) are neither read nor written.  pad: the
// rows of the padding (DenseStorage).
__device__ __forceinline__ void permute_rows(double *__restrict__ A, int n, const int32_t *perm, const uint8_t *pad) {
    constexpr int kRows = 64 * kLuWaves / 32, kPer = kLuMaxNP / kRows;
    const int tid = thread_id(), col = tid & 31, r0 = tid >> 5;
    if (!__syncthreads_or(tid < n && perm[tid] != tid)) return;
    for (int c0 = 0; c0 < n; c0 += 32) {
        const int c = c0 + col;
        double v[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int r = r0 + kRows * k, from = r < n ? perm[r] : r;
            v[k] = r < n && c < n && from < n && from != r ? A[uint32_t(from * n + c)] : 0.0;
            if (r < n && c < n && from >= n) v[k] = DenseStorage<double, true>::decode(pad[(from - n) * n + c]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int r = r0 + kRows * k;
            if (r < n && c < n && perm[r] != r) A[uint32_t(r * n + c)] = v[k];
        }
    }
}

// The workgroups resident at once take the matrices in turn, so that the scratch
// (n > 64: lu_scratch_bytes a workgroup, the inverses of the diagonal blocks of L
// and the rows of the padding) does not grow with the batch.
template <typename T>
__host__ __device__ constexpr size_t lu_inverse_elems(int NP) {
    return size_t((NP + kLuW - 1) / kLuW - 1) * kLuW * kLuW;
}
template <typename T>
__host__ __device__ constexpr size_t lu_scratch_bytes(int n, int NP) {
    return n <= kLuW ? 0 : lu_inverse_elems<T>(NP) * sizeof(T) + (size_t(NP - n) * n + 15) / 16 * 16;
}

template <typename T, bool kOneBlock>
__global__ void __launch_bounds__(64 * kLuWaves) k_lu_factor(int n, int batch, double *A0, int32_t *perm_out,
                                                             int32_t *info, unsigned char *scratch) {
    extern __shared__ double smem[];
    unsigned char *lds = reinterpret_cast<unsigned char *>(smem);
    const int NP = (n + 15) / 16 * 16;
    const LuLds<T, kLuWaves> l(NP, lds);
    const int32_t *perm = l.perm;
    T *dinv = reinterpret_cast<T *>(scratch + blockIdx.x * lu_scratch_bytes<T>(n, NP));
    // one block column: Xb is free once the panel is factored
    uint8_t *pad = reinterpret_cast<uint8_t *>(kOneBlock ? l.Xb : dinv + lu_inverse_elems<T>(NP));
    for (int m = blockIdx.x; m < batch; m += gridDim.x) {
        double *A = A0 + size_t(m) * n * n;
        lu_factor_left<T, kLuWaves, 4>(DenseStorage<T, kOneBlock>{A, n, pad, l.rwave + 3}, NP, nullptr, dinv,
                                       info ? info + m : nullptr, lds, DenseSource<T>{A, n});
        __syncthreads();
        for (int i = thread_id(); i < n; i += 64 * kLuWaves) perm_out[size_t(m) * n + i] = perm[i];
        permute_rows(A, n, perm, pad);
        __syncthreads();
    }
}

template <typename T>
static LuFactorPlan plan_factor(int n, long long batch) {
    const int NP = (n + 15) / 16 * 16;
    LuFactorPlan p;
    p.fn = n <= kLuW ? reinterpret_cast<const void *>(&k_lu_factor<T, true>)
                     : reinterpret_cast<const void *>(&k_lu_factor<T, false>);
    p.lds = lu2_lds_bytes<T, kLuWaves>(NP);
    int per_cu = 0, cus = 0, dev = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, p.fn, 64 * kLuWaves, p.lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    p.grid = int(std::min<long long>(batch, (long long)per_cu * cus));
    p.scratch = size_t(p.grid) * lu_scratch_bytes<T>(n, NP);
    return p;
}

LuFactorPlan plan_lu_factor(int n, long long batch, int prec) {
    return prec == ABDF_PREC_FP32_LU ? plan_factor<float>(n, batch) : plan_factor<double>(n, batch);
}

hipError_t launch_lu_factor(const LuFactorPlan &p, int n, long long batch, double *A, int32_t *perm, int32_t *info,
                            void *scratch, hipStream_t st) {
    int nn = n, nb = int(batch);
    void *args[] = {&nn, &nb, &A, &perm, &info, &scratch};
    return hipLaunchKernel(p.fn, dim3(unsigned(p.grid)), dim3(64 * kLuWaves), args, p.lds, st);
}

// ------------------------------------------------------------------ solve --

constexpr int kSolveThreads = 512;
constexpr int kSolveDepth = 6;   // tiles in flight

// Solves (P^T L U) z = b, LU as launch_lu_factor leaves it, z over b.  The
// factor is read once, as the stream of 64 x 64 tiles of lu_solve_left, but
// the diagonal blocks themselves are read, not inverses: a block's tile goes to
// LDS and one wave substitutes through it, a lane per row (64 steps of a
// broadcast and a multiply-add), while the tiles to come are in flight.  An
// inverse used once costs far more than it saves.  Rows begin on 8-byte
// boundaries, so 8 bytes a load: 16 lanes to a row.  Bound by the read of the
// factors (2 MB of order 500 a workgroup): 256 matrices take 0.18 ms, 600
// 0.43 ms (2.8 TB/s); through padded copies and inverses 1.07 and 1.61 ms.
template <int NB>
__global__ void __launch_bounds__(kSolveThreads) k_lu_solve(int n, const double *__restrict__ LU0, const int32_t *perm,
                                                           double *b0) {
    using Order = SolveOrder<NB>;
    constexpr int H = kLuW / 16, RP = kSolveThreads / 16, P = kLuW / RP;
    __shared__ double y[NB * kLuW], bs[NB * kLuW], t[kLuW], D[kLuW * kLdb];
    const int tid = thread_id(), lane16 = tid & 15, row16 = tid >> 4, lane = tid & 63, wave = wave_of(tid);
    const double *LU = LU0 + size_t(blockIdx.x) * n * n;
    double *b = b0 + size_t(blockIdx.x) * n;
    const int Wl = n - kLuW * (NB - 1);   // order of the last block
    double buf[kSolveDepth][P][H];
    auto load = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, ib = Order::ib(q), jb = Order::jb(q);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int rr = row16 + RP * p, r = ib * kLuW + (ib == NB - 1 ? min(rr, Wl - 1) : rr);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int cc = lane16 + 16 * h;
                buf[q % kSolveDepth][p][h] = LU[uint32_t(r * n + jb * kLuW + (jb == NB - 1 ? min(cc, Wl - 1) : cc))];
            }
        }
    };
    static_for<(kSolveDepth < Order::total ? kSolveDepth : Order::total)>([&](auto q) __attribute__((always_inline)) { load(q); });
    for (int i = tid; i < NB * kLuW; i += kSolveThreads) bs[i] = i < n ? b[i] : 0.0;
    __syncthreads();
    for (int i = tid; i < NB * kLuW; i += kSolveThreads) {
        const int from = i < n ? perm[size_t(blockIdx.x) * n + i] : i;
        y[i] = uint32_t(from) < uint32_t(NB * kLuW) ? bs[from] : 0.0;
    }
    __syncthreads();
    double acc[P] = {};
    static_for<Order::total>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, ib = Order::ib(q), jb = Order::jb(q), r0 = ib * kLuW;
        constexpr bool up = Order::up(q);
        double(&a)[P][H] = buf[q % kSolveDepth];
        if constexpr (jb != ib) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                // y is zero past n, but the entry read there is another column's
                const bool in = jb < NB - 1 || lane16 + 16 * h < Wl;
                const double yc = y[jb * kLuW + lane16 + 16 * h];
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p] = in ? fma(a[p][h], yc, acc[p]) : acc[p];
            }
        } else {
            const int W = ib == NB - 1 ? Wl : kLuW;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int r = row16 + RP * p;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int c = lane16 + 16 * h;
                    D[r * kLdb + c] = r < W && c < W ? a[p][h] : (r == c ? 1.0 : 0.0);
                }
                const double s = row_sum(acc[p]);
                acc[p] = 0.0;
                if (lane16 == 0) t[r] = r < W ? y[r0 + r] - s : 0.0;
            }
            __syncthreads();
            if (wave == 0) {
                const double *Dr = D + lane * kLdb;
                double v = t[lane];
                if constexpr (!up)
                    v = substitute<true, true, true>(Dr, 1, 1.0, v);
                else
                    v = substitute<false, false, true>(Dr, 1, Dr[lane], v);
                y[r0 + lane] = v;
            }
            __syncthreads();
        }
        if constexpr (q + kSolveDepth < Order::total) load(std::integral_constant<int, q + kSolveDepth>{});
        // the tiles in flight stay those named above
        __builtin_amdgcn_sched_barrier(0);
    });
    for (int i = tid; i < n; i += kSolveThreads) b[i] = y[i];
}

hipError_t launch_lu_solve(int n, long long batch, const double *LU, const int32_t *perm, double *b, hipStream_t st) {
#define ABDF_SOLVE(NB) \
    case NB: hipLaunchKernelGGL((k_lu_solve<NB>), dim3(unsigned(batch)), dim3(kSolveThreads), 0, st, n, LU, perm, b); break
    switch ((n + kLuW - 1) / kLuW) {
        ABDF_SOLVE(1);
        ABDF_SOLVE(2);
        ABDF_SOLVE(3);
        ABDF_SOLVE(4);
        ABDF_SOLVE(5);
        ABDF_SOLVE(6);
        ABDF_SOLVE(7);
        default: hipLaunchKernelGGL((k_lu_solve<8>), dim3(unsigned(batch)), dim3(kSolveThreads), 0, st, n, LU, perm, b); break;
    }
#undef ABDF_SOLVE
    return hipGetLastError();
}

}  // namespace abdf
