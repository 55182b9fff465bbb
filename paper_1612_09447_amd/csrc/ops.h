// Device-side views shared by the kernels: the instance map, row sums of the
// finest matrices in either storage, CSR rows.
#pragma once

#include <type_traits>

#include "eqs_internal.h"
#include "sell.h"

namespace eqs {

// ---------------------------------------------------- instances (batches)
// Independent instances occupy contiguous ranges of free rows. Every
// 256-row block of the finest level holds rows of at most two instances (each
// instance has >= 256 rows when there is more than one), so a block writes a
// pair of partial sums: [2b] for the instance of its first row, [2b+1] for the
// next instance (0 if the block lies in one instance).
struct InstMap {
    const int32_t* __restrict__ row_off;   // [n_inst + 1] first row of every instance
    const int32_t* __restrict__ blk_inst;  // [blocks] instance of each block's first row
    int32_t n_inst;
    int32_t rows1;  // the row count when n_inst == 1 (no table lookups then), else -1
    int32_t subs;   // rows per thread of a workgroup, one after the other: 1 with several instances
    int32_t nparts; // n_inst == 1: partial sums per array (part[B], not pairs) that the kernel reads
};

// B: the block's row-block index (its logical block, see row_block)
__device__ __forceinline__ void block_instances(const InstMap& m, int32_t& lo, int32_t& bound, int64_t B) {
    if (m.rows1 >= 0) {
        lo = 0;
        bound = m.rows1;
        return;
    }
    lo = m.blk_inst[B];
    bound = m.row_off[lo + 1];
}

// ---- row sums of the finest matrices, in either storage -------------------
// Op::sum(g, row, m, inst, f) is sum_j a_ij f(j) for the row of global thread g,
// `inst` the row's instance; one thread per row, workgroups of 256 rows.
template <typename T>
struct SellOp {
    static constexpr bool kScaled = true;  // as the finest smoothing operator it holds A w D^-1
    template <typename S>
    using Of = SellOp<S>;
    SellView<T> A;
    __device__ __forceinline__ int64_t block() const { return row_block(A.xcd); }
    __device__ __forceinline__ bool live(int64_t g) const { return g < (int64_t)A.n_slices * 64; }
    __device__ __forceinline__ int32_t row(int64_t g) const { return sell_perm_row<1>(A.perm, g); }
    __device__ __forceinline__ int32_t rows() const { return A.n_rows; }
    template <typename F>
    __device__ __forceinline__ T sum(int64_t g, int32_t row, const InstMap&, int32_t, F f) const {
        return sell_accum<1>(A, g, row, f);
    }
};
// By diagonals (Dia): no slice table and no column ids, so a row's 2 K + 1
// values and operands are one round of independent, contiguous loads instead of
// three dependent ones, and half of the values come from the cache (the lower
// triangle is the upper one of an earlier row): 32 B of matrix a row in FP64
// instead of 70, 16 instead of 42 in FP32. At 2.1M rows, in traces of steps on one
// card, the CG SpMV takes 40 us instead of 51 and the pre-smoother 21 instead of
// 27.5. Terms are added in column order; an absent entry (zero) adds nothing
// whatever its operand.
template <typename T, int K>
struct DiaOp {
    static constexpr bool kScaled = false;
    static constexpr int kDiagonals = K;
    template <typename S>
    using Of = DiaOp<S, K>;
    const T* __restrict__ val;
    const int32_t* __restrict__ offs;
    int32_t n;
    int32_t off[K];
    __device__ __forceinline__ int64_t block() const { return row_block(1); }
    __device__ __forceinline__ bool live(int64_t g) const { return g < n; }
    __device__ __forceinline__ int32_t row(int64_t g) const { return (int32_t)g; }
    __device__ __forceinline__ int32_t rows() const { return n; }
    // the row's values in column order, and their product
    __device__ __forceinline__ void values(int32_t row, const InstMap& m, int32_t inst, T (&v)[2 * K + 1]) const {
        const int32_t r0 = m.rows1 >= 0 ? 0 : m.row_off[inst];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t d = offs ? offs[inst * K + k] : off[k];
            const T lo = val[(int64_t)(k + 1) * n + (row - d >= r0 ? row - d : row)];
            v[K - 1 - k] = row - d >= r0 ? lo : T(0);
            v[K + 1 + k] = val[(int64_t)(k + 1) * n + row];
        }
        v[K] = val[row];
    }
    template <typename F>
    __device__ __forceinline__ T product(int32_t row, const InstMap& m, int32_t inst, const T (&v)[2 * K + 1], F f) const {
        const int32_t r0 = m.rows1 >= 0 ? 0 : m.row_off[inst];
        T x[2 * K + 1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t d = offs ? offs[inst * K + k] : off[k];
            x[K - 1 - k] = (T)f(row - d >= r0 ? row - d : row);
            x[K + 1 + k] = (T)f(row + d < n ? row + d : row);
        }
        x[K] = (T)f(row);
        T acc = T(0);
#pragma unroll
        for (int e = 0; e < 2 * K + 1; ++e) acc += v[e] == T(0) ? T(0) : v[e] * x[e];
        return acc;
    }
    template <typename F>
    __device__ __forceinline__ T sum(int64_t, int32_t row, const InstMap& m, int32_t inst, F f) const {
        T v[2 * K + 1];
        values(row, m, inst, v);
        return product(row, m, inst, v, f);
    }
};
template <typename T, int K>
static DiaOp<T, K> dia_op(const Dia<T>& D) {
    DiaOp<T, K> o{D.val, D.offs, D.n, {}};
    for (int k = 0; k < K; ++k) o.off[k] = D.off[k];
    return o;
}
// Runs the statement given last with `op` the operator in its storage.
#define EQS_WITH_OP(D, SELLVIEW, ...)                                     \
    do {                                                                   \
        if ((D).K == 3) { const auto op = dia_op<OpT, 3>(D); __VA_ARGS__; }       \
        else if ((D).K == kMaxDiagonals) { const auto op = dia_op<OpT, kMaxDiagonals>(D); __VA_ARGS__; } \
        else { const SellOp<OpT> op{SELLVIEW}; __VA_ARGS__; }                     \
    } while (0)

// By diagonals the product is with A itself and w_j r_j, w = w D^-1.
template <typename T>
__device__ __forceinline__ T presmoothed(const SellOp<T>& op, int64_t g, int32_t row, const InstMap& m, int32_t inst,
                                         const T*, const double* __restrict__ r) {
    return op.sum(g, row, m, inst, [&](int32_t j) { return (T)r[j]; });
}
template <typename T, int K>
__device__ __forceinline__ T presmoothed(const DiaOp<T, K>& op, int64_t g, int32_t row, const InstMap& m, int32_t inst,
                                         const T* __restrict__ w, const double* __restrict__ r) {
    return op.sum(g, row, m, inst, [&](int32_t j) { return w[j] * (T)r[j]; });
}

// ---- CSR with L lanes per row ---------------------------------------------
template <typename T>
struct CsrView {
    const int32_t* __restrict__ rp;
    const int32_t* __restrict__ col;
    const int16_t* __restrict__ d16;  // offsets from offset_base(row) instead of col when set
    const T* __restrict__ val;
    int32_t n_rows, n_cols;
    // offsets from the row's entry here instead when set: rows that reach further than 32767 from their
    // place but span no more than 65535 (2.1M rows, the restriction from level 1: 11.3 -> 10.3 us alone)
    const int32_t* __restrict__ rbase;
};
template <typename T>
static CsrView<T> cview(const SpMat<T>& A) {
    return CsrView<T>{A.rowptr, A.col, A.d16, A.val, A.n_rows, A.n_cols, A.rbase};
}

// Views of a level's operator with the pre-smoothing values a_ij omega / a_jj.
template <typename T>
static SellView<T> sview(const Level<T>& lv) {
    SellView<T> v = view(lv.A.sell);
    v.val = lv.sval;
    return v;
}
template <typename T>
static CsrView<T> scview(const Level<T>& lv) {
    CsrView<T> v = cview(lv.A);
    v.val = lv.sval;
    return v;
}

// Row sum of A (lanes of one group split the row), with x_j given by f(j).
template <int L, typename T, typename F>
__device__ __forceinline__ T csr_row(const CsrView<T>& A, int32_t row, int lane, F f) {
    // each lane takes entries lane, lane + L, ... of the row, U = 4 at a time:
    // positions past the row's end re-read its last entry and are dropped by a
    // select, so the loads carry no branch; the lane's sum runs in entry order.
    // (Groups of 16 for rows of 614 entries over 64 lanes, one round of loads
    // instead of three, measured slower: 12.0 against 11.4 us, the clamped
    // re-reads of the last group costing more than the rounds saved.)
    constexpr int U = 4;
    T acc = T(0);
    const int32_t end = A.rp[row + 1];
    const int32_t base = A.rbase ? A.rbase[row] : offset_base(row, A.n_rows, A.n_cols);
    for (int32_t k = A.rp[row] + lane; k < end; k += U * L) {
        T t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t kk = min(k + u * L, end - 1);
            const int32_t j = A.d16 ? base + (int32_t)A.d16[kk] : A.col[kk];
            t[u] = A.val[kk] * f(j);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc += (k + u * L < end) ? t[u] : T(0);
    }
    return group_sum<L>(acc);
}

}  // namespace eqs
