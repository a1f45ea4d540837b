// Left-looking blocked LU with partial pivoting, one workgroup per matrix
// of W waves, and the matching triangular solves.  The matrix is read through a
// source functor when each block column is first gathered, so it can be
// formed on the fly (the Newton matrix) instead of being stored first.
//
// Storage.  The matrix keeps its rows where they are: row r of P A (the
// "logical" row r) is storage row perm[r].  Pivoting only swaps entries of
// perm, so no row of the matrix is ever moved in memory; every access to a
// factor row goes through perm.  After the factorisation, storage row perm[r]
// holds row r of L (strictly lower part, unit diagonal implied) and of U.
// For each 64-row diagonal block b the inverses of its unit-lower and upper
// triangles are stored in dinv[b][0] and dinv[b][1] (64 x 64, row-major), so
// the triangular solves are products with dense blocks.
//
// Factorisation of block column j (columns 64j .. 64j + Wj - 1):
//  1. the block column is gathered (rows through perm) into MFMA accumulator
//     registers: with W waves, wave w owns row tiles w, w + W, ..., and all 4
//     column tiles of 16;
//  2. for every earlier block i: U_ij = inv(L_ii) C_i (rows 64i..64i+63 of the
//     block column, staged through LDS), then the rows below block i are
//     updated C -= L_{:,i} U_ij on the matrix cores, L read from memory;
//  3. the panel (rows >= 64j) is factored in 16-column sub-panels, one thread
//     per row.  First on the diagonal: one wave factors the sub-panel's 16 x 16
//     diagonal block without row exchanges (lane k holds row k, the pivot row
//     broadcast from its lane), then every other row eliminates against those
//     U rows with no exchange between waves; this is accepted when every
//     multiplier of the sub-panel is at most kPivotThreshold in magnitude
//     (threshold pivoting, u = 1 / kPivotThreshold: the diagonal entry is at
//     least u times the largest candidate of its column).  Otherwise the
//     sub-panel is factored again from its saved entries with partial
//     pivoting: arg-max pivot search (ties to the smaller logical row, as
//     LAPACK's idamax), scaling and rank-1 update; rows keep their positions
//     and only their logical labels change.  After each sub-panel the rest of
//     the block column is updated on the matrix cores;
//  4. the inverses of the diagonal block's triangles are formed and stored,
//     and the block column is written back through perm.
#pragma once

#include "device_common.hpp"
#include "device_lu.hpp"

namespace abdf {

constexpr int kLuW = 64;          // block-column width
constexpr int kLuMaxNP = 512;     // one thread per row in the panel
// Largest multiplier with which a sub-panel keeps its diagonal pivots.  On the
// Newton matrices I - c J of the chemistry networks fewer than 1% of the
// sub-panels exceed it (at large c, late in an integration); the factors'
// backward error stays at the level of partial pivoting there.
constexpr double kPivotThreshold = 4.0;

// The factorisation runs on W waves, W * 64 >= NP (one thread per row in the
// panel); each wave holds row tiles w, w + W, ... of the block column in at most
// lu_slots accumulator tiles.
template <int W>
constexpr int lu_slots = kLuMaxNP / 16 / (W >= 8 ? W : 8);
constexpr int lu_wave_bits(int w) { return w <= 1 ? 0 : 1 + lu_wave_bits(w / 2); }
constexpr int kLdb = 65;          // LDS leading dimension of 64-wide staging buffers

template <typename T>
struct V4;
template <>
struct V4<double> { typedef double type __attribute__((ext_vector_type(4))); };
template <>
struct V4<float> { typedef float type __attribute__((ext_vector_type(4))); };

// lane group and accumulator register holding row t (0..15) of a 16x16 tile
template <typename T>
__device__ inline int tile_row_group(int t);
template <>
__device__ inline int tile_row_group<double>(int t) { return t & 3; }
template <>
__device__ inline int tile_row_group<float>(int t) { return t >> 2; }
template <typename T>
__device__ inline int tile_row_reg(int t);
template <>
__device__ inline int tile_row_reg<double>(int t) { return t >> 2; }
template <>
__device__ inline int tile_row_reg<float>(int t) { return t & 3; }

// LDS layout of lu_factor_left (element type T for the staging region).
constexpr int kPanLd = 17;        // row stride of the 16-column sub-panel buffer
constexpr int kU12Ld = 49;        // row stride of the 16 x 48 sub-panel U block
constexpr int kCrowLd = 17;       // candidate pivot row: 16 entries and the pivot's reciprocal
// rows of the staging buffers of a block column (64, or the matrix's order)
__host__ __device__ constexpr int lu2_stage_rows(int NP) { return NP < kLuW ? NP : kLuW; }
template <typename T>
__host__ __device__ constexpr size_t lu2_work_elems(int NP) {
    const size_t panel = size_t(NP) * kPanLd + 16 * kU12Ld;
    const size_t stage = 3 * size_t(lu2_stage_rows(NP)) * kLdb + (sizeof(T) == 4 ? 1536 : 0);
    return panel > stage ? panel : stage;
}
template <typename T, int W>
__host__ __device__ constexpr size_t lu2_lds_bytes(int NP) {
    return 5 * size_t(NP) * sizeof(int32_t)                        // perm, sto, pos_log, log_pos, pidx
           + kLuW * sizeof(int32_t)                                // piv_pos
           + 2 * W * (sizeof(double) + sizeof(int32_t))     // arg-max partials, double-buffered
           + 16 + 18 * sizeof(int32_t)                                // row flags; diagonal positions, flag
           + 2 * W * kCrowLd * sizeof(T)                    // candidate pivot rows, double-buffered
           + 16 * kCrowLd * sizeof(T)                                 // factored diagonal block
           + lu2_work_elems<T>(NP) * sizeof(T) + 64;
}

// Its parts.  After a factorisation of one block column (NP <= 64) perm, Xb
// (inverse of the unit-lower triangle) and Ub (of the upper one) stay valid.
template <typename T, int W>
struct LuLds {
    int32_t *perm;      // logical row -> storage row
    int32_t *sto;       // position -> storage row (this block column)
    int32_t *pos_log;   // position -> logical row
    int32_t *log_pos;   // logical row -> position
    int32_t *pidx;      // position -> pivot column in this block, or -1
    int32_t *piv_pos;   // pivot column -> position
    double *redv;       // [2][waves] arg-max partials
    int32_t *redi;
    int32_t *rwave;     // [2] wave holding logical row r; first zero pivot (1-based) or INT_MAX; DenseStorage::nan
    int32_t *dpos;      // [16] positions of the diagonal pivot rows
    int32_t *spec_bad;  // the diagonal pivots were refused
    T *crow;            // [2][waves][kCrowLd] candidate rows
    T *Db;              // [16][kCrowLd] factored diagonal block
    T *Cb, *Ub, *Xb;    // [64][kLdb] each (rows: lu2_stage_rows); Cb: left-looking, inverses
    __device__ __forceinline__ LuLds(int NP, unsigned char *smem) {
        perm = reinterpret_cast<int32_t *>(smem);
        sto = perm + NP;
        pos_log = sto + NP;
        log_pos = pos_log + NP;
        pidx = log_pos + NP;
        piv_pos = pidx + NP;
        redv = reinterpret_cast<double *>(piv_pos + kLuW);
        redi = reinterpret_cast<int32_t *>(redv + 2 * W);
        rwave = redi + 2 * W;
        dpos = rwave + 4;
        spec_bad = dpos + 16;
        crow = reinterpret_cast<T *>(dpos + 18);
        Db = crow + 2 * W * kCrowLd;
        Cb = Db + 16 * kCrowLd;
        Ub = Cb + lu2_stage_rows(NP) * kLdb;
        Xb = Ub + lu2_stage_rows(NP) * kLdb;
    }
};

// Orders one wave's LDS accesses before and after this point as written: the
// LDS executes a wave's instructions in issue order, so a value one lane
// writes is seen by every lane of the wave that reads it later; only the
// compiler must be kept from moving the accesses (no instruction is emitted).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Leading dimension of the stored factors: rows 4 kB apart would put a block
// column's rows in the same few channels of the L2 and of the memory.  (Slots::lda
// is NP itself where not even one slot fits otherwise.)
constexpr int lu_ld(int NP) { return NP % 128 == 0 ? NP + 16 : NP; }

// Elements of the per-matrix inverse diagonal blocks.
template <typename T>
__host__ __device__ constexpr size_t lu2_dinv_elems(int NP) {
    return size_t((NP + kLuW - 1) / kLuW) * 2 * kLuW * kLuW;
}

// Inverses of the unit-lower and the upper triangle of the W x W diagonal block
// held in LDS (leading dimension kLdb), written to D[0] and D[1] (64 x 64
// row-major, global), block-recursively on 16 x 16 blocks: the diagonal
// blocks by substitution (the first half of the threads for inv(L), the second
// for inv(U), one lane per column), then the off-diagonal blocks level by
// level on the matrix cores, one wave per block,
// X_ij = -X_ii sum_k L_ik X_kj (lower) and Y_ij = -Y_ii sum_k U_ik Y_kj (upper).
// Xb, Yb: W x kLdb LDS outputs; Tb: 1536 elements of LDS scratch (FP32 only).  Every
// thread of the workgroup must call this (it contains barriers).  Without kUpper
// only the lower one.
template <typename T, int NW, bool kUpper>
__device__ __forceinline__ void diag_inverses(const T *Cb, int W, T *D, T *Xb, T *Yb, T *Tb) {
    constexpr int HALF = 32 * NW;   // threads of each triangle
    const int tid = thread_id();
    const bool upper = tid >= HALF;
    const int h = tid % HALF;
    const int nb = W / 16;
    T *Z = upper ? Yb : Xb;
    T *Tz = Tb + (upper ? 768 : 0);
    // zero the outputs (rows of the block; the rest is not read)
    for (int e = h; e < 64 * W; e += HALF) Z[(e >> 6) * kLdb + (e & 63)] = T(0);
    __syncthreads();
    // diagonal 16 x 16 blocks: one lane per column, the column's entries in
    // registers, by substitution (no barrier, no shuffle); lanes h < 64 of
    // each half, lane h holding column h of the 64 x 64 block (fewer lanes take
    // several columns in turn)
    for (int hc = h; hc < 64; hc += HALF) {
        const int b = hc >> 4, kc = hc & 15;
        if (b < nb && (kUpper || !upper)) {
            const T *Bd = Cb + 16 * b * kLdb + 16 * b;     // the diagonal block, leading dimension kLdb
            double xs[16];
            if (!upper) {
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    double acc = 0.0;
#pragma unroll
                    for (int m = 0; m < t; ++m) {
                        const double p = double(Bd[t * kLdb + m]) * xs[m];
                        acc = m >= kc ? acc + p : acc;
                    }
                    xs[t] = t < kc ? 0.0 : (t == kc ? 1.0 : -acc);
                }
            } else {
#pragma unroll
                for (int t = 15; t >= 0; --t) {
                    double acc = 0.0;
#pragma unroll
                    for (int m = t + 1; m < 16; ++m) {
                        const double p = double(Bd[t * kLdb + m]) * xs[m];
                        acc = m <= kc ? acc + p : acc;
                    }
                    const double d = double(Bd[t * kLdb + t]);
                    xs[t] = t > kc ? 0.0 : (t == kc ? 1.0 / d : -acc / d);
                }
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) Z[(16 * b + t) * kLdb + 16 * b + kc] = T(xs[t]);
        }
    }
    __syncthreads();
    // off-diagonal blocks, by distance from the diagonal, one wave per block on
    // the matrix cores: the sum over the blocks between, then the product with
    // the diagonal block's inverse (lower X_ij = -X_ii sum_{k=j..i-1} L_ik X_kj,
    // upper Y_ij = -Y_ii sum_{k=i+1..j} U_ik Y_kj)
    {
        using Mt = Mfma<T>;
        using acc_t = typename Mt::acc_t;
        const int wave = wave_of(tid), lane = tid & 63, lr = lane & 15, lg = lane >> 4;
        for (int d = 1; d < nb; ++d) {
            for (int blk = wave; blk < (kUpper ? 2 : 1) * (nb - d); blk += NW) {
                const bool up = blk >= nb - d;
                const int bi = up ? blk - (nb - d) : blk;
                const int i = up ? bi : bi + d, jb = up ? bi + d : bi;
                const int k0 = up ? i + 1 : jb;
                T *Zt = up ? Yb : Xb;
                acc_t acc = acc_t{0, 0, 0, 0};
                for (int kb = 0; kb < d; ++kb) {
                    const int k = k0 + kb;
#pragma unroll
                    for (int st = 0; st < 4; ++st)
                        acc = Mt::mma(Cb[(16 * i + lr) * kLdb + 16 * k + 4 * st + lg],
                                      Zt[(16 * k + 4 * st + lg) * kLdb + 16 * jb + lr], acc);
                }
                acc_t acc2 = acc_t{0, 0, 0, 0};
                if constexpr (sizeof(T) == sizeof(double)) {
                    // the accumulator's register st holds rows 4 st + lane / 16:
                    // the B operand of step st as it stands
#pragma unroll
                    for (int st = 0; st < 4; ++st)
                        acc2 = Mt::mma(Zt[(16 * i + lr) * kLdb + 16 * i + 4 * st + lg], acc[st], acc2);
                } else {
                    T *Ts = Tb + 256 * blk;
#pragma unroll
                    for (int v = 0; v < 4; ++v) Ts[Mt::row(lane, v) * 16 + lr] = acc[v];
                    wave_lds_order();
#pragma unroll
                    for (int st = 0; st < 4; ++st)
                        acc2 = Mt::mma(Zt[(16 * i + lr) * kLdb + 16 * i + 4 * st + lg], Ts[(4 * st + lg) * 16 + lr],
                                       acc2);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) Zt[(16 * i + Mt::row(lane, v)) * kLdb + 16 * jb + lr] = -acc2[v];
            }
            __syncthreads();
        }
    }
    if (kUpper || !upper)
        for (int e = h; e < 64 * W; e += HALF) D[(upper ? kLuW * kLuW : 0) + e] = Z[(e >> 6) * kLdb + (e & 63)];
}

// The value v of lane src (the same on every lane), on every lane.
__device__ __forceinline__ double lane_value(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_value(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// Where lu_factor_left keeps the factors: rows in storage order, leading
// dimension lda, in T (a slot's own storage).
template <typename T>
struct SlotStorage {
    static constexpr bool kKeepInverses = true;   // the solves use them
    T *A;
    int lda;
    using v4 = typename V4<T>::type;
    __device__ __forceinline__ void begin_column() {}
    __device__ __forceinline__ static bool is_pad(int) { return false; }
    __device__ __forceinline__ static void store_pad(int, int, T) {}
    // four entries of a row from column c, a multiple of 4
    __device__ __forceinline__ v4 load4(int row, int c) const {
        return *reinterpret_cast<const v4 *>(A + uint32_t(row * lda + c));
    }
    __device__ __forceinline__ void store(int row, int c, T v) const { A[uint32_t(row * lda + c)] = v; }
};

// The caller's n x n FP64 matrix itself, factored in place.  The rows that pad it
// to a multiple of 16 (the identity's, zero in its columns) go to pad, n entries
// each: a column that is zero or NaN in every row left may take one as its pivot.
// Their entries stay zeros of either sign or, beside a factor that is not finite,
// become NaN, so a byte says which (as doubles they took the scratch of 256
// matrices of order 500 past 64 MiB, whose allocation cost 0.3 ms a call).  Only
// once one is NaN (nan: an LDS flag) are they read back.  The padding's columns are
// not stored.  Rows begin on 8-byte boundaries.  kOneBlock (n <= 64): nothing is
// read back, and pad is in the LDS.
template <typename T, bool kOneBlock>
struct DenseStorage {
    static constexpr bool kKeepInverses = false;
    double *A;
    int n;
    uint8_t *pad;
    int32_t *nan;
    bool read_pad = false;
    using v4 = typename V4<T>::type;
    __device__ __forceinline__ static double decode(int code) {
        return code == 2 ? std::numeric_limits<double>::quiet_NaN() : (code == 1 ? -0.0 : 0.0);
    }
    // before a block column, after a barrier
    __device__ __forceinline__ void begin_column() { read_pad = __builtin_amdgcn_readfirstlane(*nan) != 0; }
    __device__ __forceinline__ v4 load4(int row, int c) const {
        double d[4];
        __builtin_memcpy(d, A + uint32_t(min(row, n - 1) * n + c), sizeof(d));
        v4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = row < n ? T(d[k]) : T(0);
        if (!kOneBlock && read_pad && row >= n) {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = T(decode(pad[(row - n) * n + c + k]));
        }
        return v;
    }
    __device__ __forceinline__ void store(int row, int c, T v) const {
        if (row < n && c < n) A[uint32_t(row * n + c)] = double(v);
    }
    __device__ __forceinline__ bool is_pad(int row) const { return row >= n; }
    __device__ __forceinline__ void store_pad(int row, int c, T v) const {
        if (row >= n && c < n) {
            pad[(row - n) * n + c] = v != v ? 2 : (signbit(v) ? 1 : 0);
            if (v != v) *nan = 1;
        }
    }
};

// The entries of the matrix to factor (storage row, column).  A source yields an
// entry in two steps: row(r, c0), what the lanes of row r need for the 64
// columns from c0 (a multiple of 64), and entry(that, r, col), so that the
// gather can issue every row's loads before the entry loads that depend on
// them.
template <typename T>
struct DenseSource {
    const double *A;
    int n;
    struct Row { int32_t off; };
    __device__ __forceinline__ Row row(int r, int) const { return {min(r, n - 1) * n}; }
    __device__ __forceinline__ T entry(const Row &w, int r, int col) const {
        const double v = A[uint32_t(w.off + min(col, n - 1))];
        return r < n && col < n ? T(v) : T(r == col ? 1.0 : 0.0);
    }
};

// Factors the matrix whose entries src yields (read once, when its block
// column is gathered) into st, which needs no initial contents.  Leaves the row
// order in LuLds::perm as well as in perm_out [NP] (null: only there).  dinv: the
// inverse diagonal blocks; unless the storage keeps them for solves, only those
// of L that later block columns need, one 64 x 64 block after the other.  A single
// wave (W = 1) holds kTiles x kTiles tiles, NP <= 16 kTiles.
template <typename T, int W, int kTiles, typename Src, typename Storage>
__device__ __forceinline__ void lu_factor_left(Storage st, int NP, int32_t *__restrict__ perm_out,
                                               T *__restrict__ dinv, int32_t *info, unsigned char *smem,
                                               const Src &src) {
    using M = Mfma<T>;
    using acc_t = typename M::acc_t;
    using v4 = typename V4<T>::type;
    constexpr bool kKeep = Storage::kKeepInverses;
    constexpr int kSlots = W == 1 ? kTiles : lu_slots<W>, kCT = W == 1 ? kTiles : 4;
    constexpr int kDinvStride = (kKeep ? 2 : 1) * kLuW * kLuW;
    const int tid0 = thread_id();
    const int RT = NP / 16;
    const int NB = (NP + kLuW - 1) / kLuW;

    const LuLds<T, W> lds(NP, smem);
    int32_t *perm = lds.perm, *sto = lds.sto, *pos_log = lds.pos_log, *log_pos = lds.log_pos, *pidx = lds.pidx;
    int32_t *piv_pos = lds.piv_pos, *redi = lds.redi, *rwave = lds.rwave, *dpos = lds.dpos, *spec_bad = lds.spec_bad;
    double *redv = lds.redv;
    T *crow = lds.crow, *Db = lds.Db, *Cb = lds.Cb, *Ub = lds.Ub, *Xb = lds.Xb;
    T *P = Cb;                                             // [NP][kPanLd] (panel)
    T *U12 = P + size_t(NP) * kPanLd;                      // [16][kU12Ld]

    for (int i = tid0; i < NP; i += (64 * W)) perm[i] = i;
    if (tid0 < 16) dpos[tid0] = 0;      // every position read from it stays in the panel
    if (tid0 == 0) {
        rwave[2] = 0x7fffffff;
        rwave[3] = 0;
    }
    __syncthreads();

    for (int j = 0; j < NB; ++j) {
        // anew for each block column: the accumulators need the registers that
        // its many LDS addresses would take
        const int tid = thread_id(), lane = tid & 63, wave = wave_of(tid);
        const int g = lane >> 4, lc = lane & 15;
        const int c0 = j * kLuW;
        st.begin_column();
        const int Wj = min(kLuW, NP - c0);
        const int CTj = Wj / 16;
        for (int q = tid; q < NP; q += (64 * W)) {
            sto[q] = perm[q];
            pos_log[q] = q;
            log_pos[q] = q;
            pidx[q] = -1;
        }
        acc_t acc[kSlots][kCT];
        // 1. gather the block column (positions = logical rows at this point):
        //    what each of the lane's rows needs first, then every entry, so
        //    that each lane has all its row loads in flight together and then
        //    all its entry loads (the accumulators are not live yet).  Tiles
        //    outside the matrix read column c0 + lc of row 0 and are zeroed.
        {
            typename Src::Row rw[kSlots][4];
            int srow[kSlots][4];
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
#pragma unroll
                for (int v = 0; v < 4; ++v) srow[s][v] = rt < RT ? perm[16 * rt + M::row(lane, v)] : 0;
            }
#pragma unroll
            for (int s = 0; s < kSlots; ++s)
#pragma unroll
                for (int v = 0; v < 4; ++v) rw[s][v] = src.row(srow[s][v], c0);
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
#pragma unroll
                for (int ct = 0; ct < kCT; ++ct)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const T val = src.entry(rw[s][v], srow[s][v], c0 + 16 * (ct < CTj ? ct : 0) + lc);
                        acc[s][ct][v] = (rt < RT && ct < CTj) ? val : T(0);
                    }
            }
        }
        // 2. updates from the earlier block columns.  What comes from memory is
        //    asked for ahead of the barriers and the products it would
        //    otherwise wait behind: the inverse of L_ii before C_i is staged,
        //    this wave's first tile of L before U_ij is complete, each further
        //    tile before the products with the one before it.
#pragma unroll 1
        for (int i = 0; i < j; ++i) {
            const int r0 = i * kLuW;
            const T *Li = dinv + size_t(i) * kDinvStride;   // inverse of the unit-lower block i
            // the 16 tiles of U_ij = inv(L_ii) C_i, spread over all waves (a
            // workgroup of fewer than four waves has one block column)
            constexpr int TPW = W >= 4 ? 16 / W : 1;
            const int t0 = wave * TPW, tr = t0 >> 2;
            v4 ia[4];
            if constexpr (W >= 4) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    ia[kk] = *reinterpret_cast<const v4 *>(Li + (16 * tr + lc) * kLuW + 16 * kk + 4 * g);
            }
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
                if (rt >= 4 * i && rt < 4 * i + 4) {
#pragma unroll
                    for (int ct = 0; ct < kCT; ++ct)
                        if (ct < CTj)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                Cb[(16 * (rt - 4 * i) + M::row(lane, v)) * kLdb + 16 * ct + lc] = acc[s][ct][v];
                }
            }
            __syncthreads();
            // rows of the first tile below block i that this wave holds
            v4 la[4];
            auto load_tile = [&](int rt) {
                const int row = perm[16 * rt + lc];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) la[kk] = st.load4(row, r0 + 16 * kk + 4 * g);
            };
            {
                const int below = 4 * (i + 1);
                const int first = wave >= below ? wave : wave + (below - wave + W - 1) / W * W;
                if (first < RT) load_tile(first);
            }
            if constexpr (W >= 4) {
#pragma unroll
                for (int k = 0; k < TPW; ++k) {
                    const int ct = (t0 + k) & 3;
                    if (ct < CTj) {
                        acc_t u = acc_t{0, 0, 0, 0};
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                u = M::mma(ia[kk][e], Cb[(16 * kk + 4 * g + e) * kLdb + 16 * ct + lc], u);
#pragma unroll
                        for (int v = 0; v < 4; ++v) Ub[(16 * tr + M::row(lane, v)) * kLdb + 16 * ct + lc] = u[v];
                    }
                }
            }
            __syncthreads();
            // the rows of block i take their tiles of U_ij; the rows below are
            // updated C -= L_{:,i} U_ij
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
                if (rt >= 4 * i && rt < 4 * i + 4) {
                    const int tr = rt - 4 * i;
#pragma unroll
                    for (int ct = 0; ct < kCT; ++ct)
                        if (ct < CTj)
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[s][ct][v] = Ub[(16 * tr + M::row(lane, v)) * kLdb + 16 * ct + lc];
                }
                if (rt >= 4 * (i + 1) && rt < RT) {
                    v4 a[4];
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) a[kk] = la[kk];
                    if (rt + W < RT) load_tile(rt + W);
                    if (CTj == 4) {
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
#pragma unroll
                                for (int ct = 0; ct < kCT; ++ct)
                                    acc[s][ct] = M::mma(-a[kk][e], Ub[(16 * kk + 4 * g + e) * kLdb + 16 * ct + lc],
                                                        acc[s][ct]);
                    } else {
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
#pragma unroll
                                for (int ct = 0; ct < (kCT < 3 ? kCT : 3); ++ct)
                                    if (ct < CTj)
                                        acc[s][ct] = M::mma(-a[kk][e], Ub[(16 * kk + 4 * g + e) * kLdb + 16 * ct + lc],
                                                            acc[s][ct]);
                    }
                }
            }
            __syncthreads();
        }
        // 3. panel factorisation, 16-column sub-panels.  Rows stay at their
        //    positions; pivoting assigns logical rows to positions.  First on the
        //    diagonal, as long as it is accepted: then no row has been exchanged
        //    in this block column, position and logical row are the same, the
        //    pivot rows of sub-panel sp are row tile 4 j + sp and the unused rows
        //    the tiles below.  Unrolled, so that a sub-panel's column tile is a
        //    constant of the accumulators.  The first sub-panel refused and those
        //    after it go through the general loop below.  (The panel phases
        //    of a 500-species factorisation: 16.4 us a sub-panel through the
        //    general loop alone, timed over a batch of 256 matrices; 9.7 this
        //    way, timed inside a solve of 512 cells.)
        int from = CTj;      // the first sub-panel left to the general loop
        static_for<kCT>([&](auto spc) __attribute__((always_inline)) {
            constexpr int sp = decltype(spc)::value;
            if (sp >= from) return;
            const int tid = thread_id(), lane = tid & 63, wave = wave_of(tid);
            const int g = lane >> 4, lc = lane & 15;
            const int dt = 4 * j + sp, rb = 16 * dt;
            // (a) the sub-panel's column tile to LDS, one row per position (the
            //     accumulators keep it until (c))
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
                if (rt >= dt && rt < RT)
#pragma unroll
                    for (int v = 0; v < 4; ++v) P[(16 * rt + M::row(lane, v)) * kPanLd + lc] = acc[s][sp][v];
            }
            if (tid == 0) spec_bad[0] = 0;
            __syncthreads();
            // (b1) the diagonal block, rows rb .. rb + 15
            if (wave == 0) {
                // the 16 x 16 block in registers; column c: every entry below row
                // c takes its multiplier or its update from row c, each lane
                // reading what it needs from the lanes that hold it before it
                // changes its own; the factored block then goes to Db.  A pivot
                // below the smallest normal number refuses the diagonal (partial
                // pivoting then forms such multipliers by division).
                bool bad = false;
                if constexpr (sizeof(T) == sizeof(float)) {
                    // FP32: lane i < 16 holds row i; the pivot and the rest of
                    // row c reach every lane by readlane
                    T a[16];
                    const bool row_lane = lane < 16;
#pragma unroll
                    for (int c = 0; c < 16; ++c) a[c] = P[(rb + (row_lane ? lane : 0)) * kPanLd + c];
                    T uii = T(1);
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const T piv = lane_value(a[c], c);
                        const bool normal = fabs(piv) >= std::numeric_limits<T>::min();
                        const T rinv = T(1) / (normal ? piv : T(1));
                        if (lane == c) uii = a[c];
                        const bool below = row_lane && lane > c;
                        const T l = a[c] * rinv;
                        bad |= !normal;
                        bad |= below && !(fabs(l) <= T(kPivotThreshold));
#pragma unroll
                        for (int j = c + 1; j < 16; ++j) {
                            const T ucj = lane_value(a[j], c);
                            if (below) a[j] = a[j] - l * ucj;
                        }
                        if (below) a[c] = l;
                    }
                    if (row_lane) {
#pragma unroll
                        for (int c = 0; c < 16; ++c) Db[lane * kCrowLd + c] = a[c];
                        Db[lane * kCrowLd + 16] = T(1) / uii;   // used only when every pivot is normal
                    }
                } else {
                    // FP64 (fewer registers): lane l holds the entries of rows
                    // i = 4 t + l / 16 (t = 0..3) in column j = l % 16.  A column
                    // is a chain of its pivot (readlane), its reciprocal and the
                    // multipliers (a row broadcast each); the pivot row's entries
                    // come by LDS permutes meanwhile.
                    const int jj = lane & 15, gg = lane >> 4;
                    T a[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) a[t] = P[(rb + 4 * t + gg) * kPanLd + jj];
                    static_for<16>([&](auto cc) __attribute__((always_inline)) {
                        constexpr int c = decltype(cc)::value, tc = c >> 2, gc = c & 3;
                        const T ucj = __shfl(a[tc], 16 * gc + jj);
                        const T piv = lane_value(a[tc], 16 * gc + c);
                        const bool normal = fabs(piv) >= std::numeric_limits<T>::min();
                        const T rinv = T(1) / (normal ? piv : T(1));
                        T l[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) l[t] = row_broadcast<c>(a[t]) * rinv;
                        bad |= !normal;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int i = 4 * t + gg;
                            if (4 * t + 3 > c) {
                                const bool below = i > c;
                                bad |= below && jj == c && !(fabs(l[t]) <= T(kPivotThreshold));
                                const T upd = a[t] - l[t] * ucj;
                                a[t] = below && jj == c ? l[t] : (below && jj > c ? upd : a[t]);
                            }
                        }
                    });
#pragma unroll
                    for (int t = 0; t < 4; ++t) Db[(4 * t + gg) * kCrowLd + jj] = a[t];
                    wave_lds_order();
                    if (lane < 16) Db[lane * kCrowLd + 16] = T(1) / Db[lane * kCrowLd + lane];   // used only when every pivot is normal
                }
                if (__ballot(bad) != 0 && lane == 0) spec_bad[0] = 1;
            }
            __syncthreads();
            // (b2) every row below, one thread each, against the diagonal block's
            //      U rows (no exchange between waves), the result written over
            //      the row in LDS.  A U row is read once per wave, an entry a
            //      lane, and its entries handed round as scalars: read from LDS
            //      by every lane they took its whole rate.
            const int q = tid;
            const bool row = q >= rb + 16 && q < NP;
            {
                bool bad = false;
                if (64 * wave + 63 >= rb + 16 && 64 * wave < NP) {
                    T x[16];
                    const int qr = row ? q : rb;      // idle lanes work on a row of the panel for nothing
#pragma unroll
                    for (int c = 0; c < 16; ++c) x[c] = P[qr * kPanLd + c];
                    T un = Db[lane < 17 ? lane : 0];
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const T u = un;
                        if (c < 15) un = Db[(c + 1) * kCrowLd + (lane < 17 ? lane : 0)];
                        const T l = x[c] * lane_value(u, 16);
                        bad |= !(fabs(l) <= T(kPivotThreshold));
                        x[c] = l;
#pragma unroll
                        for (int cb = c + 1; cb < 16; ++cb) x[cb] -= l * lane_value(u, cb);
                    }
                    if (row) {
#pragma unroll
                        for (int c = 0; c < 16; ++c) P[q * kPanLd + c] = x[c];
                    }
                }
                if (__ballot(bad && row) != 0 && lane == 0) spec_bad[0] = 1;
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(spec_bad[0]) != 0) {
                from = sp;
                return;
            }
            // accepted: the diagonal rows are the pivots, labels unchanged
            if (q >= rb && q < rb + 16) {
                pidx[q] = 16 * sp + (q - rb);
                piv_pos[16 * sp + (q - rb)] = q;
            }
            // (c) back to the accumulators; (d) the pivot rows of the remaining
            //     column tiles of the block to LDS
            const int nct = CTj - sp - 1;
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
                if (rt >= dt && rt < RT) {
                    const T *src = rt == dt ? Db : P + 16 * rt * kPanLd;
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[s][sp][v] = src[M::row(lane, v) * kPanLd + lc];
                    if (rt == dt) {
#pragma unroll
                        for (int ct = sp + 1; ct < kCT; ++ct)
                            if (ct < CTj)
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    U12[M::row(lane, v) * kU12Ld + 16 * (ct - sp - 1) + lc] = acc[s][ct][v];
                    }
                }
            }
            if constexpr (sp < 3) {
                if (nct == 0) return;
                __syncthreads();
                // U12 of the pivot rows, a column a thread
                if (tid < 16 * nct) {
                    T u[16];
#pragma unroll
                    for (int i2 = 0; i2 < 16; ++i2) u[i2] = U12[i2 * kU12Ld + tid];
#pragma unroll
                    for (int i2 = 1; i2 < 16; ++i2) {
#pragma unroll
                        for (int m = 0; m < i2; ++m) u[i2] -= Db[i2 * kCrowLd + m] * u[m];
                    }
#pragma unroll
                    for (int i2 = 0; i2 < 16; ++i2) U12[i2 * kU12Ld + tid] = u[i2];
                }
                __syncthreads();
                // the rows below
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const int rt = wave + W * s;
                    if (rt > dt && rt < RT) {
                        T a[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[e] = -P[(16 * rt + lc) * kPanLd + 4 * e + g];
#pragma unroll
                        for (int ct = sp + 1; ct < kCT; ++ct)
                            if (ct < CTj)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    acc[s][ct] = M::mma(a[e], U12[(4 * e + g) * kU12Ld + 16 * (ct - sp - 1) + lc],
                                                        acc[s][ct]);
                    }
                    if (rt == dt) {
#pragma unroll
                        for (int ct = sp + 1; ct < kCT; ++ct)
                            if (ct < CTj)
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    acc[s][ct][v] = U12[M::row(lane, v) * kU12Ld + 16 * (ct - sp - 1) + lc];
                    }
                }
                __syncthreads();
            }
        });
        __syncthreads();
        // the general loop, from the first sub-panel whose diagonal was refused
#pragma unroll 1
        for (int sp = from; sp < CTj; ++sp) {
            // (a) the sub-panel's column tile to LDS, one row per position (the
            //     accumulators keep it until (c), so it can be written again)
            auto panel_to_lds = [&]() {
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const int rt = wave + W * s;
                    if (rt >= 4 * j && rt < RT)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            T val = acc[s][0][v];
#pragma unroll
                            for (int ct = 1; ct < kCT; ++ct)
                                if (ct == sp) val = acc[s][ct][v];
                            P[(16 * rt + M::row(lane, v)) * kPanLd + lc] = val;
                        }
                }
            };
            panel_to_lds();
            // (b) one thread per position factors the 16 columns.  Each
            //     thread knows the logical row of its position (mylog).
            const int q = tid;
            bool active = q >= c0 && q < NP && pidx[q] < 0;
            const bool participated = active;
            int mylog = active ? pos_log[q] : 0x7fffffff;
            // (b1) diagonal pivots: the rows of logical index rb .. rb + 15
            const int rb = c0 + 16 * sp;
            const bool is_diag = active && mylog >= rb && mylog < rb + 16;
            if (tid == 0) spec_bad[0] = 0;
            if (is_diag) dpos[mylog - rb] = q;
            __syncthreads();
            if (wave == 0) {
                // the 16 x 16 diagonal block in registers; column c: every entry
                // below row c takes its multiplier or its update from row c,
                // each lane reading what it needs from the lanes that hold it
                // before it changes its own; the factored block then goes to Db.
                // A pivot below the smallest normal number refuses the diagonal
                // (partial pivoting then forms such multipliers by division).
                bool bad = false;
                if constexpr (sizeof(T) == sizeof(float)) {
                    // FP32: lane i < 16 holds row i; the pivot and the rest of
                    // row c reach every lane by readlane
                    T a[16];
                    const bool row_lane = lane < 16;
#pragma unroll
                    for (int c = 0; c < 16; ++c) a[c] = P[dpos[row_lane ? lane : 0] * kPanLd + c];
                    T uii = T(1);
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const T piv = lane_value(a[c], c);
                        const bool normal = fabs(piv) >= std::numeric_limits<T>::min();
                        const T rinv = T(1) / (normal ? piv : T(1));
                        if (lane == c) uii = a[c];
                        const bool below = row_lane && lane > c;
                        const T l = a[c] * rinv;
                        bad |= !normal;
                        bad |= below && !(fabs(l) <= T(kPivotThreshold));
#pragma unroll
                        for (int j = c + 1; j < 16; ++j) {
                            const T ucj = lane_value(a[j], c);
                            if (below) a[j] = a[j] - l * ucj;
                        }
                        if (below) a[c] = l;
                    }
                    if (row_lane) {
#pragma unroll
                        for (int c = 0; c < 16; ++c) Db[lane * kCrowLd + c] = a[c];
                        Db[lane * kCrowLd + 16] = T(1) / uii;   // used only when every pivot is normal
                    }
                } else {
                    // FP64 (fewer registers): lane l holds the entries of rows
                    // i = 4 t + l / 16 (t = 0..3) in column j = l % 16, read by
                    // shuffles
                    const int jj = lane & 15, gg = lane >> 4;
                    T a[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) a[t] = P[dpos[4 * t + gg] * kPanLd + jj];
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const int tc = c >> 2, gc = c & 3;
                        const T piv = __shfl(a[tc], 16 * gc + c);
                        const bool normal = fabs(piv) >= std::numeric_limits<T>::min();
                        const T rinv = T(1) / (normal ? piv : T(1));
                        const T ucj = __shfl(a[tc], 16 * gc + jj);
                        T l[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) l[t] = __shfl(a[t], 16 * gg + c) * rinv;
                        bad |= !normal;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int i = 4 * t + gg;
                            if (i > c) {
                                if (jj == c) {
                                    bad |= !(fabs(l[t]) <= T(kPivotThreshold));
                                    a[t] = l[t];
                                } else if (jj > c) {
                                    a[t] = a[t] - l[t] * ucj;
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) Db[(4 * t + gg) * kCrowLd + jj] = a[t];
                    wave_lds_order();
                    if (lane < 16) Db[lane * kCrowLd + 16] = T(1) / Db[lane * kCrowLd + lane];   // used only when every pivot is normal
                }
                if (__ballot(bad) != 0 && lane == 0) spec_bad[0] = 1;
            }
            __syncthreads();
            // (b2) every other unpivoted row against the diagonal block's U
            //      rows (the elimination of the partial-pivoting loop below
            //      with its pivots fixed, so no exchange between waves), the
            //      result written over the row in LDS; the diagonal rows take
            //      their factored entries
            {
                bool bad = false;
                if (active && !is_diag) {
                    T x[16];
#pragma unroll
                    for (int c = 0; c < 16; ++c) x[c] = P[q * kPanLd + c];
#pragma unroll
                    for (int c = 0; c < 16; ++c) {
                        const T *urow = Db + c * kCrowLd;
                        const T l = x[c] * urow[16];
                        bad |= !(fabs(l) <= T(kPivotThreshold));
                        x[c] = l;
#pragma unroll
                        for (int cb = c + 1; cb < 16; cb += 4) {
                            T uv[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (cb + u < 16) uv[u] = urow[cb + u];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (cb + u < 16) x[cb + u] -= l * uv[u];
                        }
                        // the U rows are the same for every row: keep the
                        // scheduler from hoisting all their loads at once
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int c = 0; c < 16; ++c) P[q * kPanLd + c] = x[c];
                } else if (is_diag) {
                    const int k = mylog - rb;
#pragma unroll
                    for (int c = 0; c < 16; ++c) P[q * kPanLd + c] = Db[k * kCrowLd + c];
                }
                if (__ballot(bad) != 0 && lane == 0) spec_bad[0] = 1;
            }
            __syncthreads();
            if (spec_bad[0] == 0) {
                // accepted: the diagonal rows are the pivots, labels unchanged
                if (is_diag) {
                    pidx[q] = 16 * sp + (mylog - rb);
                    piv_pos[16 * sp + (mylog - rb)] = q;
                }
                __syncthreads();
            } else {
            // (b3) refused: the sub-panel again from the accumulators, with
            //      partial pivoting.  The winner of the pivot search among a
            //      wave's lanes publishes its row, so one barrier per column
            //      suffices.  A wave without unpivoted rows only takes part in
            //      the barriers.
            panel_to_lds();
            __syncthreads();
            const bool busy = __ballot(active) != 0;
            if (!busy && lane == 0) {
                redv[wave] = -1.0;
                redv[W + wave] = -1.0;
            }
            T x[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) x[c] = active ? P[q * kPanLd + c] : T(0);
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const int gc = 16 * sp + c;
                const int r = c0 + gc;
                const int buf = c & 1;
                if (busy) {
                    const double ax = fabs(double(x[c]));
                    double bv = (active && ax == ax) ? ax : -1.0;   // NaN never wins
                    int bl = mylog;
                    wave_argmax_ballot(bv, bl);
                    if (lane == 0) { redv[buf * W + wave] = bv; redi[buf * W + wave] = bl; }
                    if (active && mylog == r) rwave[buf] = wave;
                    // the wave's candidate row (or row r, kept when nothing is
                    // finite) with the reciprocal of its entry in column c, or 0
                    // where that is below the smallest normal number (then the
                    // multipliers are formed by division, as LAPACK does)
                    if (active && mylog == (bv < 0.0 ? r : bl)) {
                        T *cr = crow + (buf * W + wave) * kCrowLd;
#pragma unroll
                        for (int cc = c; cc < 16; ++cc) cr[cc] = x[cc];
                        cr[16] = fabs(x[c]) >= std::numeric_limits<T>::min() ? T(1) / x[c] : T(0);
                    }
                }
                __syncthreads();
                if (!busy) continue;
                // cross-wave arg-max: lane w < 8 holds wave w's partial; ties go
                // to the smaller logical row
                int lp, wv;
                {
                    const double fv = lane < W ? redv[buf * W + lane] : -2.0;
                    const int fi = lane < W ? redi[buf * W + lane] : 0x7fffffff;
                    double m = dpp_max_step<0xB1, 0xf>(fv);    // quad_perm [1,0,3,2]
                    m = dpp_max_step<0x4E, 0xf>(m);            // quad_perm [2,3,0,1]
                    m = dpp_max_step<0x141, 0xf>(m);           // row_half_mirror: lanes 0..7 hold their max
                    if (W > 8) m = dpp_max_step<0x140, 0xf>(m);   // row_mirror: lanes 0..15
                    {
                        const int lo = __builtin_amdgcn_readlane(__double2loint(m), 0);
                        const int hi = __builtin_amdgcn_readlane(__double2hiint(m), 0);
                        m = __hiloint2double(hi, lo);
                    }
                    if (m < 0.0) {          // no finite candidate: keep logical row r
                        lp = r;
                        wv = rwave[buf];
                    } else {
                        const unsigned long long hit = __ballot(lane < W && fv == m);
                        if (__popcll(hit) == 1) {
                            wv = __ffsll(static_cast<unsigned long long>(hit)) - 1;
                            lp = __builtin_amdgcn_readlane(fi, wv);
                        } else {
                            double tv = (lane < W && fv == m) ? 1.0 : -1.0;
                            int tk = (lane < W && fv == m) ? (fi << lu_wave_bits(W)) + lane : 0x7fffffff;
                            wave_argmax(tv, tk);
                            lp = tk >> lu_wave_bits(W);
                            wv = tk & (W - 1);
                        }
                    }
                }
                const T *urow = crow + (buf * W + wv) * kCrowLd;
                const T piv = urow[c];
                const T rinv = urow[16];
                if (lane == 0 && piv == T(0)) atomicMin(&rwave[2], r + 1);
                if (active) {
                    if (mylog == lp) {               // this position becomes logical row r
                        mylog = r;
                        active = false;
                        pidx[q] = gc;
                        piv_pos[gc] = q;
                    } else {
                        if (mylog == r) mylog = lp;  // row r moves to the pivot's old logical index
                        T l;
                        if (rinv != T(0))
                            l = x[c] * rinv;
                        else
                            l = piv != T(0) ? x[c] / piv : x[c];
                        x[c] = l;
                        // the pivot row in groups of four entries, each group's
                        // loads issued together before its updates
#pragma unroll
                        for (int cb = c + 1; cb < 16; cb += 4) {
                            T uv[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (cb + u < 16) uv[u] = urow[cb + u];
                            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);   // the group's LDS reads
                            __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);   // then VALU
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                if (cb + u < 16) x[cb + u] -= l * uv[u];
                        }
                    }
                }
            }
            if (participated) {
#pragma unroll
                for (int c = 0; c < 16; ++c) P[q * kPanLd + c] = x[c];
                pos_log[q] = mylog;
            }
            __syncthreads();
            }   // partial pivoting
            // (c) back to the accumulators
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const int rt = wave + W * s;
                if (rt >= 4 * j && rt < RT)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const T val = P[(16 * rt + M::row(lane, v)) * kPanLd + lc];
#pragma unroll
                        for (int ct = 0; ct < kCT; ++ct)
                            if (ct == sp) acc[s][ct][v] = val;
                    }
            }
            // (d) the remaining column tiles of the block: U12 of this
            //     sub-panel's pivot rows, then the update of unused rows
            if (sp + 1 < CTj) {
                const int nct = CTj - sp - 1;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const int rt = wave + W * s;
                    if (rt >= 4 * j && rt < RT)
#pragma unroll
                        for (int ct = 1; ct < kCT; ++ct)
                            if (ct > sp && ct < CTj)
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int pi = pidx[16 * rt + M::row(lane, v)] - 16 * sp;
                                    if (pi >= 0 && pi < 16)
                                        U12[pi * kU12Ld + 16 * (ct - sp - 1) + lc] = acc[s][ct][v];
                                }
                }
                __syncthreads();
                if (tid < 16 * nct) {
                    T u[16];
#pragma unroll
                    for (int i2 = 0; i2 < 16; ++i2) u[i2] = U12[i2 * kU12Ld + tid];
#pragma unroll
                    for (int i2 = 1; i2 < 16; ++i2) {
                        const T *Lr = P + piv_pos[16 * sp + i2] * kPanLd;
#pragma unroll
                        for (int m = 0; m < i2; ++m) u[i2] -= Lr[m] * u[m];
                    }
#pragma unroll
                    for (int i2 = 0; i2 < 16; ++i2) U12[i2 * kU12Ld + tid] = u[i2];
                }
                __syncthreads();
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const int rt = wave + W * s;
                    if (rt >= 4 * j && rt < RT) {
                        const bool unused = pidx[16 * rt + lc] < 0;
                        T a[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[e] = unused ? -P[(16 * rt + lc) * kPanLd + 4 * e + g] : T(0);
#pragma unroll
                        for (int ct = 1; ct < kCT; ++ct) {
                            if (ct > sp && ct < CTj) {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    acc[s][ct] = M::mma(a[e], U12[(4 * e + g) * kU12Ld + 16 * (ct - sp - 1) + lc],
                                                        acc[s][ct]);
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int pi = pidx[16 * rt + M::row(lane, v)] - 16 * sp;
                                    if (pi >= 0 && pi < 16) acc[s][ct][v] = U12[pi * kU12Ld + 16 * (ct - sp - 1) + lc];
                                }
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
        // the last sub-panel's rows are read back from P before the staging
        // buffer below (which shares P's memory) is written
        __syncthreads();
        for (int q2 = tid; q2 < NP; q2 += (64 * W))
            if (q2 >= c0) perm[pos_log[q2]] = sto[q2];
        // 4. diagonal block (logical rows c0 .. c0 + Wj - 1) to LDS, its
        //    triangles' inverses, and the block column back to its storage rows
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const int rt = wave + W * s;
            if (rt >= 4 * j && rt < RT)
#pragma unroll
                for (int ct = 0; ct < kCT; ++ct)
                    if (ct < CTj)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int lr = pos_log[16 * rt + M::row(lane, v)] - c0;
                            if (lr >= 0 && lr < Wj) Cb[lr * kLdb + 16 * ct + lc] = acc[s][ct][v];
                        }
        }
        // the block column goes back first, so that the accumulators are free
        // while the inverses are formed
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const int rt = wave + W * s;
            if (rt < RT)
#pragma unroll
                for (int ct = 0; ct < kCT; ++ct)
                    if (ct < CTj)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            st.store(sto[16 * rt + M::row(lane, v)], c0 + 16 * ct + lc, acc[s][ct][v]);
            // the rows of the padding: one wave has them, unless rows were exchanged
            int row[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) row[v] = rt < RT ? sto[16 * rt + M::row(lane, v)] : 0;
            if (__any(st.is_pad(max(max(row[0], row[1]), max(row[2], row[3]))))) {
#pragma unroll
                for (int ct = 0; ct < kCT; ++ct)
                    if (ct < CTj)
#pragma unroll
                        for (int v = 0; v < 4; ++v) st.store_pad(row[v], c0 + 16 * ct + lc, acc[s][ct][v]);
            }
        }
        __syncthreads();
        if (kKeep || j + 1 < NB) {
            diag_inverses<T, W, kKeep>(Cb, Wj, dinv + size_t(j) * kDinvStride, Xb, Ub, Xb + lu2_stage_rows(NP) * kLdb);
            __syncthreads();
        }
    }
    if (perm_out)
        for (int i = tid0; i < NP; i += (64 * W)) perm_out[i] = perm[i];
    if (tid0 == 0 && info) *info = rwave[2] == 0x7fffffff ? 0 : rwave[2];
}

// The order in which a solve reads the tiles of a factor of NB block rows: per
// block row of L (downwards), then of U (upwards), its tiles off the diagonal
// from left to right, then the inverse of its diagonal block's triangle.
template <int NB>
struct SolveOrder {
    static constexpr int total = NB * (NB + 1);
    static constexpr bool up(int q) { return q >= total / 2; }
    static constexpr int row(int q) {   // block rows done before tile q's
        int e = q % (total / 2), m = 0;
        while (e > m) e -= ++m;
        return m;
    }
    static constexpr int ib(int q) { return up(q) ? NB - 1 - row(q) : row(q); }
    static constexpr int jb(int q) {    // == ib: the diagonal block's inverse
        const int e = q % (total / 2) - row(q) * (row(q) + 1) / 2;
        return up(q) ? (e < row(q) ? ib(q) + 1 + e : ib(q)) : e;
    }
};

// Solves (P^T L U) z = b for one matrix factored by lu_factor_left, with the
// NT threads of a workgroup.  Row r of the factors is storage row perm[r] (LDS);
// y starts as b[perm[.]].  b[NP] (LDS, FP64) is read, the solution is left in y[NP] (LDS); t is
// 64 doubles of LDS scratch.  Factor entries are widened to FP64; the
// arithmetic is FP64.
// N (even, 64 (NB - 1) < N <= NP) is the order of the padded matrix: its rows
// and columns from N on are the identity's, in the matrix and so in its factors
// (no pivot is taken from them before column N), and b is zero there; the
// products then stop at N and y keeps its zeros past N.
//
// The factor is read once as a stream of 64 x 64 tiles.  No tile's address
// depends on a result, so each thread keeps its parts of the next kDepth tiles
// in flight in registers while it works on the current one: one workgroup
// alone must draw what its compute unit can (kDepth x 32 kB in FP64 against
// some 2 us of latency), where loads issued block by block wait for every
// block's reductions and barriers.  The stream is unrolled (NB is a constant):
// a tile is then its loads at constant offsets from its rows' addresses, its
// products with solution entries held in registers, and nothing else.  With the
// position in the stream computed at run time the bookkeeping took longer
// than the loads: 19.3 us a solve of 200 species against 12.7, 69 against 64 of
// 500 with 256 cells at once; block by block it was 26.8 and 115 us.  What is
// left is the chain of two reductions and two barriers a block row (some
// 0.7 us) at 200 species, and at 500 the memory as well (2.3 MB a solve).
// 16 lanes to a row, 16 bytes (VW entries) a load.
template <typename T, int NT, int NB, int kDepth>
__device__ __forceinline__ void lu_solve_left(const T *__restrict__ A, int lda, const T *__restrict__ dinv,
                                              const int32_t *perm, int NP, int N,
                                              const double *b, double *y, double *t) {
    using Order = SolveOrder<NB>;
    constexpr int VW = 16 / int(sizeof(T));          // factor entries per 16-byte load
    constexpr int H = kLuW / (16 * VW);              // loads per row of a tile
    constexpr int RP = NT / 16, P = kLuW / RP;       // rows per pass, rows per thread
    const int tid = thread_id();
    const int lane16 = tid & 15, row16 = tid >> 4;
    const int Wl = N - kLuW * (NB - 1);              // rows of the last block
    for (int i = tid; i < NP; i += NT) y[i] = b[perm[i]];
    // where this thread's rows of each block row begin, at its first column
    // (rows past the end read the last one again)
    uint32_t off[NB][P];
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int rr = row16 + RP * p, r = ib * kLuW + (ib == NB - 1 ? min(rr, Wl - 1) : rr);
            off[ib][p] = uint32_t(perm[r]) * uint32_t(lda) + VW * lane16;
        }
    T buf[kDepth][P][H][VW];
    // The zero side of a triangle's inverse is not read: a column there loads the
    // 16 bytes that hold the diagonal instead (a cache line the row needs
    // anyway) and contributes nothing.
    auto load = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        constexpr int ib = Order::ib(q), jb = Order::jb(q);
        constexpr bool up = Order::up(q), last = ib == NB - 1;
        T(&dst)[P][H][VW] = buf[q % kDepth];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const T *src;
                if constexpr (jb == ib) {
                    const int rr = last ? min(row16 + RP * p, Wl - 1) : row16 + RP * p;
                    const int c = VW * lane16 + 16 * VW * h, dq = rr & ~(VW - 1);
                    src = dinv + (ib * 2 + (up ? 1 : 0)) * (kLuW * kLuW) + uint32_t(rr * kLuW + (up ? max(c, dq) : min(c, dq)));
                } else if constexpr (jb == NB - 1) {
                    // the last block column may be narrower
                    const int c = jb * kLuW + VW * lane16 + 16 * VW * h;
                    src = A + (off[ib][p] - VW * lane16 + min(c, NP - VW));
                } else {
                    src = A + off[ib][p] + (jb * kLuW + 16 * VW * h);
                }
                __builtin_memcpy(dst[p][h], __builtin_assume_aligned(src, 16), 16);
            }
    };
    double yv[NB][H][VW];     // this lane's columns of the solution so far
    double acc[P] = {};
    auto use = [&](auto qc) __attribute__((always_inline)) {
        // products and sums exactly as written
#pragma clang fp contract(off)
        constexpr int q = decltype(qc)::value;
        constexpr int ib = Order::ib(q), jb = Order::jb(q), r0 = ib * kLuW;
        constexpr bool up = Order::up(q), last = ib == NB - 1;
        T(&a)[P][H][VW] = buf[q % kDepth];
        if constexpr (jb != ib) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                // FP32 entries past N (at most three, within the row) meet zeros of y
                const bool in = jb < NB - 1 || VW * lane16 + 16 * VW * h < Wl;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    double s;
                    s = fma(double(a[p][h][0]), yv[jb][h][0], double(a[p][h][1]) * yv[jb][h][1]);
                    if constexpr (VW == 4)
                        s = s + fma(double(a[p][h][2]), yv[jb][h][2], double(a[p][h][3]) * yv[jb][h][3]);
                    if (in) acc[p] += s;
                }
            }
            return;
        }
        const int W = last ? Wl : kLuW;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const double s = row_sum(acc[p]);
            acc[p] = 0.0;
            const int r = row16 + RP * p;
            if (lane16 == 0 && r < W) t[r] = y[r0 + r] - s;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int c = VW * lane16 + 16 * VW * h;
            if (c < W) {
                double tv[VW];
#pragma unroll
                for (int k = 0; k < VW; ++k) tv[k] = c + k < W ? t[c + k] : 0.0;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int r = min(row16 + RP * p, W - 1);
                    double term[VW];
#pragma unroll
                    for (int k = 0; k < VW; ++k) {
                        const bool in = c + k < W && (up ? c + k >= r : c + k <= r);
                        term[k] = in ? double(a[p][h][k]) * tv[k] : 0.0;
                    }
                    if constexpr (VW == 2)
                        acc[p] += term[0] + term[1];
                    else
                        acc[p] += (term[0] + term[1]) + (term[2] + term[3]);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const double s = row_sum(acc[p]);
            acc[p] = 0.0;
            const int r = row16 + RP * p;
            if (lane16 == 0 && r < W) y[r0 + r] = s;
        }
        __syncthreads();
        // the block's entries for the block rows to come
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int k = 0; k < VW; ++k) {
                const int c = VW * lane16 + 16 * VW * h + k;
                yv[ib][h][k] = y[r0 + (last ? min(c, NP - r0 - 1) : c)];
            }
    };
    static_for<(kDepth < Order::total ? kDepth : Order::total)>([&](auto q) __attribute__((always_inline)) { load(q); });
    __syncthreads();
    static_for<Order::total>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        use(qc);
        if constexpr (q + kDepth < Order::total) load(std::integral_constant<int, q + kDepth>{});
        // the tiles in flight stay those named above
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The same for any order: NB = ceil(N / 64).
template <typename T, int NT, int kDepth>
__device__ __forceinline__ void lu_solve_left(const T *__restrict__ A, int lda, const T *__restrict__ dinv,
                                              const int32_t *perm, int NP, int N,
                                              const double *b, double *y, double *t) {
#define ABDF_SOLVE(NB) \
    case NB: lu_solve_left<T, NT, NB, kDepth>(A, lda, dinv, perm, NP, N, b, y, t); break
    switch ((N + kLuW - 1) / kLuW) {
        ABDF_SOLVE(1);
        ABDF_SOLVE(2);
        ABDF_SOLVE(3);
        ABDF_SOLVE(4);
        ABDF_SOLVE(5);
        ABDF_SOLVE(6);
        ABDF_SOLVE(7);
        default: lu_solve_left<T, NT, 8, kDepth>(A, lda, dinv, perm, NP, N, b, y, t); break;
    }
#undef ABDF_SOLVE
}


// One wave's substitution through a 64 x 64 triangle, a lane per unknown: the
// unknowns k in ascending (kAscending) or descending order, w_k = v_k / d_k
// (kUnit: v_k), then v_i -= e_i[k stride] w_k for the lanes i still to come.  e, d:
// this lane's entries and its diagonal entry.  A quotient is formed from the
// pivot's reciprocal, taken by every lane at once, with one correction by its
// remainder (Markstein 1990: the rounded quotient) instead of a division in the
// chain (kDivide: by division).  kApart: a lane's products are summed apart and taken from v once, where
// it is used; where they are small beside v (a Newton matrix's diagonal is the
// largest entry) that is one rounding of v in place of up to 63.
template <bool kAscending, bool kUnit, bool kApart, bool kDivide>
__device__ __forceinline__ double substitute_lanes(const double *e, int stride, double d, double v) {
    const int lane = thread_id() & 63;
    const double rd = kUnit || kDivide ? 1.0 : 1.0 / d;
    double sum = 0.0;
#pragma unroll 8
    for (int s = 0; s < kLuW; ++s) {
        const int k = kAscending ? s : kLuW - 1 - s;
        const double r = kApart ? v - sum : v;
        const double q = r * rd, w = kUnit ? r : (kDivide ? r / d : fma(fma(-d, q, r), rd, q));
        const double x = lane_value(w, k), ek = e[k * stride];
        const bool after = kAscending ? lane > k : lane < k;
        if constexpr (kApart) {
            const double upd = fma(ek, x, sum);
            sum = lane == k ? 0.0 : (after ? upd : sum);
            v = lane == k ? w : v;
        } else {
            const double upd = fma(-ek, x, v);
            v = lane == k ? w : (after ? upd : v);
        }
    }
    return v;
}

// The same for any d and v.  The corrected quotient makes a NaN of what a division
// keeps finite or infinite: the reciprocal of a pivot below 2^-1024 or of zero is
// infinite, a quotient may pass the range, a pivot or v may be infinite.  A block
// whose unknowns do not all come out finite is done again by division.
template <bool kAscending, bool kUnit, bool kApart>
__device__ __forceinline__ double substitute(const double *e, int stride, double d, double v) {
    const double w = substitute_lanes<kAscending, kUnit, kApart, false>(e, stride, d, v);
    if constexpr (!kUnit)
        if (__ballot(!isfinite(w)) != 0) return substitute_lanes<kAscending, kUnit, kApart, true>(e, stride, d, v);
    return w;
}

// Solves M^T z = b from the factors of P M = L U (M^T = U^T L^T P): forward
// substitution with U^T, back substitution with L^T, then z[rowmap[i]] = v[i].
// The off-diagonal blocks enter as column products (lane i & 63 owns column
// i of the current 64-column block, the waves split the rows, so each wave
// reads 64 consecutive entries of a row); the diagonal blocks are solved by
// substitution (one wave, column by column, the block staged in LDS) rather
// than by their stored inverses: the reverse sweep of the BDF map amplifies
// solve errors strongly, and substitution keeps them at the level of a
// backward-stable solver.  b, z, t (>= (1 + W) * kLuW doubles) and Db
// (kLuW * kLdb doubles) are in LDS; b is consumed.
//
// A chain of block rows, each a round of loads and 64 dependent steps of one
// wave.  The row map is in LDS (in z, which is written last), so no load waits
// for another; a block's tile is asked for with its products; and no division is
// in the chain (substitute).  (The solves of a gradient of 64 cells of 200 species: 30 ms a workgroup before, 13.5 now.)
template <typename T, int W>
__device__ __forceinline__ void lu_solve_left_T(const T *__restrict__ A, int lda, const int32_t *__restrict__ rowmap, int NP,
                                                double *b, double *z, double *t, double *Db) {
    static_assert(64 * W >= kLuMaxNP, "one thread per row");
    constexpr int kU = kLuW / W;          // rows of a block per wave
    const int tid = thread_id();
    const int col = tid & 63, grp = wave_of(tid);
    const int NB = (NP + kLuW - 1) / kLuW;
    int32_t *perm = reinterpret_cast<int32_t *>(z);
    if (tid < NP) perm[tid] = rowmap[tid];
    __syncthreads();
    // one block row: wave 0 gets b[r0 + col] - sum_{r in [rb, re)} A[r][r0 + col] b[r],
    // Db the diagonal block
    auto block = [&](int r0, int Wb, int rb, int re) __attribute__((always_inline)) {
        const int cc = r0 + min(col, Wb - 1);
        double d[kU], acc = 0.0;
#pragma unroll
        for (int u = 0; u < kU; ++u) d[u] = double(A[uint32_t(perm[r0 + min(grp + W * u, Wb - 1)] * lda + cc)]);
#pragma unroll 2
        for (int q = rb; q < re; q += kLuW) {
            double a[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) a[u] = double(A[uint32_t(perm[min(q + grp + W * u, re - 1)] * lda + cc)]);
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int r = q + grp + W * u;
                if (r < re) acc += a[u] * b[r];
            }
        }
        t[kLuW + grp * kLuW + col] = acc;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int rr = grp + W * u;
            Db[rr * kLdb + col] = rr < Wb && col < Wb ? d[u] : (rr == col ? 1.0 : 0.0);
        }
        __syncthreads();
        double sum = 0.0;
        if (grp == 0) {
#pragma unroll
            for (int g = 1; g <= W; ++g) sum += t[g * kLuW + col];
            sum = col < Wb ? b[r0 + col] - sum : 0.0;
        }
        return sum;
    };
    // U^T w = b: w_k = t_k / U_kk, then t_i -= U_ki w_k for i > k  (w kept in b)
    for (int ib = 0; ib < NB; ++ib) {
        const int r0 = ib * kLuW, Wb = min(kLuW, NP - r0);
        double tv = block(r0, Wb, 0, r0);
        if (grp == 0) {
            tv = substitute<true, false, false>(Db + col, kLdb, Db[col * kLdb + col], tv);
            if (col < Wb) b[r0 + col] = tv;
        }
        __syncthreads();
    }
    // L^T v = w (unit diagonal): v_k = t_k, then t_i -= L_ki v_k for i < k  (v kept in b)
    for (int ib = NB - 1; ib >= 0; --ib) {
        const int r0 = ib * kLuW, Wb = min(kLuW, NP - r0);
        double tv = block(r0, Wb, r0 + Wb, NP);
        if (grp == 0) {
            tv = substitute<false, true, false>(Db + col, kLdb, 1.0, tv);
            if (col < Wb) b[r0 + col] = tv;
        }
        __syncthreads();
    }
    const int to = tid < NP ? perm[tid] : 0;
    const double v = tid < NP ? b[tid] : 0.0;
    __syncthreads();
    if (tid < NP) z[to] = v;
    __syncthreads();
}

}  // namespace abdf
