// SELL rows on the device: slices of one wavefront (64 lanes) each, stored
// in pairs of entries: lane l of a wavefront finds its entries 2 k and 2 k + 1 at
// sptr[s] + 128 k + 2 l, so one load fetches two values (8 or 16 bytes a lane)
// and one their columns; the slice is as wide as its longest row, rounded up to
// a pair. With L lanes
// per row a slice holds 64 / L rows: lane l serves row 64 s / L + l / L and
// takes the row's entries l % L, l % L + L, ... (long rows of coarse AMG
// operators then need 1/L as many sequential loads); the L partial sums are
// combined by cross-lane shuffles.
// Column ids are either absolute (col, 32-bit) or, when every stored entry
// lies within 32767 of offset_base(row), 16-bit offsets from it (d16): 6
// instead of 8 bytes per FP32 entry, 10 instead of 12 per FP64 entry. Where rows
// reach further (the transfers of large meshes: several planes of nodes), the
// offsets are from a base of each pair of entries (pbase), whose 128 columns lie
// close together: rows of a slice are neighbours (2.1M rows,
// FP32: the first restriction 20.5 -> 17.8 us, [G Q] 23.2 -> 21.2; they read 6 bytes
// an entry instead of 8).
// Padding entries carry value 0 and an in-range column.
#pragma once

#include <hip/hip_runtime.h>

#include "eqs_internal.h"

namespace eqs {

// ---- sums over lanes ------------------------------------------------------
// The value of the lane that the DPP control names, in the rows of 16 lanes of the
// mask (0 in the others and where there is no such lane). DPP is part of the
// vector instruction; a shuffle goes through LDS: some 100 cycles a step, and a CU's
// wavefronts share its one LDS port (CG SpMV of 266,000 rows, 36 double steps a
// wavefront: 8.9 instead of 11.0 us).
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int dpp_move(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(dpp_move<CTRL, ROWS>(__float_as_int(v)));
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_move(double v) {
    return __hiloint2double(dpp_move<CTRL, ROWS>(__double2hiint(v)), dpp_move<CTRL, ROWS>(__double2loint(v)));
}

// Sum over the L lanes of an aligned lane group (result in every lane).
template <int L, typename T>
__device__ __forceinline__ T group_sum(T v) {
    if (L > 1) v += dpp_move<0xb1>(v);   // quad_perm 1 0 3 2
    if (L > 2) v += dpp_move<0x4e>(v);   // quad_perm 2 3 0 1
    if (L > 4) v += dpp_move<0x141>(v);  // mirror in 8 lanes, whose quads are uniform by now
    if (L > 8) v += dpp_move<0x140>(v);  // mirror in 16
#pragma unroll
    for (int off = 16; off < L; off <<= 1) v += __shfl_xor(v, off, L);
    return v;
}

// Sum over the wavefront, whose lanes are all active: in lane 63, or (wave_sum) in
// every lane.
__device__ __forceinline__ double wave_total(double v) {
    v = group_sum<16>(v);
    v += dpp_move<0x142, 0xa>(v);         // row_bcast 15: rows 1 and 3 add the row before
    return v + dpp_move<0x143, 0xc>(v);   // row_bcast 31: rows 2 and 3 add rows 0 and 1
}
__device__ __forceinline__ double wave_sum(double v) {
    v = wave_total(v);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Row blocks of the sparse kernels. The hardware deals the workgroups of a
// launch to its 8 XCDs round-robin (workgroup i to XCD i mod 8). In the XCD
// order (an operator's `xcd` flag) workgroup i takes row block
// xcd_block(i, nb), so each XCD walks one contiguous range of row blocks and
// the vector entries its rows gather meet in that XCD's L2 instead of being
// fetched by several L2s. On the 2.1M-DOF workload this cut the counted
// traffic of the finest level's kernels (CG SpMV 267 -> 232 MB per launch,
// pre-smoother 168 -> 133 MB, post-smoother 177 -> 158 MB) and their times
// (post-smoother 26.7 -> 25.1 us), while the transfer products between the
// finest two levels and the level-1 smoother became slower (the restriction
// 22.9 -> 24.3 us), so M and the finest level's operator take the XCD order
// and the others the natural one. Partial sums are indexed by row block
// either way.
__device__ __forceinline__ int64_t xcd_block(int64_t i, int64_t nb) {
    const int64_t q = nb >> 3, r = nb & 7, x = i & 7;
    return x * q + (x < r ? x : r) + (i >> 3);
}
__device__ __forceinline__ int64_t row_block(int32_t xcd) {
    return xcd ? xcd_block(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
}

// The row served by global thread g of a SELL kernel with L lanes per row.
template <int L>
__device__ __forceinline__ int32_t sell_row_of(int64_t g) {
    return (int32_t)((g >> 6) * (64 / L) + ((g & 63) / L));
}

template <typename T>
struct SellView {
    const int32_t* __restrict__ sptr;
    const int32_t* __restrict__ col;
    const int16_t* __restrict__ d16;
    const T* __restrict__ val;
    int32_t n_rows, n_slices, n_cols;
    const uint8_t* __restrict__ perm;  // row order within each 256-thread window, or NULL (see sell_perm_row)
    int32_t xcd;                       // block order of its products (see row_block)
    const int32_t* __restrict__ pbase; // d16 is relative to it, pair by pair, when set
};

template <typename T>
static inline SellView<T> view(const Sell<T>& A) {
    return SellView<T>{A.sptr, A.col, A.d16, A.val, A.n_rows, A.n_slices, A.n_cols, A.perm, A.xcd, A.pbase};
}

// With a row order (perm), the rows served by one 256-thread window (4
// slices, 256 / L rows) are stored longest first, so the slices of the window
// pad less; position k of the window serves row window_base + perm[k]. The
// kernels that use it write only rows of their own window (products y = A x,
// the CG SpMV and residual, the finest smoothers), so the rows of a workgroup,
// and with them its partial sums, are the same with and without it.
template <int L>
__device__ __forceinline__ int32_t sell_perm_row(const uint8_t* __restrict__ perm, int64_t g) {
    const int32_t pos = sell_row_of<L>(g);
    if (!perm) return pos;
    const int32_t base = (int32_t)((g >> 8) * (256 / L));
    return base + (int32_t)perm[pos];
}

template <typename V>
struct Pair {
    V a, b;
};
// Pairs carry the nontemporal hint: the operator is read once per product, and
// the caches are left to the gathered vector.
template <typename V>
__device__ __forceinline__ Pair<V> load_pair(const V* __restrict__ p) {
    typedef V V2 __attribute__((ext_vector_type(2)));
    const V2 v = __builtin_nontemporal_load(reinterpret_cast<const V2*>(p));
    return Pair<V>{v.x, v.y};
}

// acc + the terms of N pairs at entry offset `at`: all loads, then all gathers,
// are in flight together.
template <int N, typename T, typename F>
__device__ __forceinline__ T sell_pairs(const SellView<T>& A, int64_t at, int32_t base, F f, T acc) {
    Pair<T> v[N];
    Pair<int32_t> j[N];
    if (A.pbase) {
        const int32_t* pb = A.pbase + __builtin_amdgcn_readfirstlane((int32_t)(at >> 7));
#pragma unroll
        for (int u = 0; u < N; ++u) {
            v[u] = load_pair(A.val + at + 128 * u);
            const Pair<int16_t> d = load_pair(A.d16 + at + 128 * u);
            const int32_t b = pb[u];
            j[u] = Pair<int32_t>{b + d.a, b + d.b};
        }
    } else if (A.d16) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            v[u] = load_pair(A.val + at + 128 * u);
            const Pair<int16_t> d = load_pair(A.d16 + at + 128 * u);
            j[u] = Pair<int32_t>{base + d.a, base + d.b};
        }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            v[u] = load_pair(A.val + at + 128 * u);
            j[u] = load_pair(A.col + at + 128 * u);
        }
    }
    T t[2 * N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        t[2 * u] = v[u].a * f(j[u].a);
        t[2 * u + 1] = v[u].b * f(j[u].b);
    }
#pragma unroll
    for (int u = 0; u < 2 * N; ++u) acc += t[u];
    return acc;
}

// sum_k a_{row,k} f(col_k) over the stored entries of `row` served by global
// thread g (rows past n_rows but inside the last slice see padding only).
// Entries are taken in groups of U whose loads are in flight together (a row of
// w stored entries costs about w / U dependent rounds of loads, then gathers;
// short rows want a small U, long ones a large U); the slice's width is the same
// for the whole wavefront, so the last, shorter group is a branch and nothing is
// loaded twice. Each lane sums in k order; with L > 1 the lane sums are then
// combined by group_sum (every lane of the group gets the row's sum).
template <int L, int U = 8, typename T, typename F>
__device__ __forceinline__ T sell_accum(const SellView<T>& A, int64_t g, int32_t row, F f) {
    const int32_t s = __builtin_amdgcn_readfirstlane((int32_t)(g >> 6));
    const int32_t beg = A.sptr[s];
    int32_t w = (A.sptr[s + 1] - beg) >> 7;  // pairs
    int64_t at = beg + 2 * (int32_t)(g & 63);
    const int32_t base = A.d16 ? offset_base(row, A.n_rows, A.n_cols) : 0;
    T acc = T(0);
    for (; w >= U / 2; w -= U / 2, at += 64 * U) acc = sell_pairs<U / 2>(A, at, base, f, acc);
    if (U > 8 && w >= 4) {
        acc = sell_pairs<4>(A, at, base, f, acc);
        w -= 4;
        at += 512;
    }
    if (w == 3) acc = sell_pairs<3>(A, at, base, f, acc);
    else if (w == 2) acc = sell_pairs<2>(A, at, base, f, acc);
    else if (w == 1) acc = sell_pairs<1>(A, at, base, f, acc);
    return group_sum<L>(acc);
}

template <int L, int U = 8, typename T, typename TX>
__device__ __forceinline__ T sell_row(const SellView<T>& A, int64_t g, int32_t row, const TX* __restrict__ x) {
    return sell_accum<L, U>(A, g, row, [&](int32_t j) { return (T)x[j]; });
}

// One lane per row (thread index = row).
template <typename T, typename TX>
__device__ __forceinline__ T sell_row(const SellView<T>& A, int32_t row, const TX* __restrict__ x) {
    return sell_row<1>(A, row, row, x);
}

}  // namespace eqs
