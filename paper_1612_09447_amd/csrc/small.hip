// CG solves of small single systems in one launch.
//
// A system of a few thousand rows spends its CG iterations on launches and on
// the chains of dependent loads at each kernel's start (30 us an iteration of
// 567 rows in seven launches, 5 us of them arithmetic and traffic). Here one
// workgroup runs the whole solve (Sec. II, Sec. V: AMG-preconditioned CG on M):
// the start residual, every iteration with its V-cycle, the check of the true
// residual and the restarts, with r, z and the coarse vectors in LDS and x, p, q
// in registers, so that an iteration is five phases between barriers:
//   b_1 = Q^T r,  x_1 = B b_1,  z = G r + Q x_1 (with r.z, r.z_old),
//   q = M z + beta q, p = z + beta p (with p.q),  x += alpha p, r -= alpha q.
// What bounds it is latency: of the loads of operators from the L2 (about 0.3 us
// each, rows' extents before their entries) and of the sums over the workgroup. So
// the operators of the folded cycle (upload_folded with the dense bottom at level
// 1) are copied to LDS once where they fit (Stage), rows by diagonals are held in
// registers, and sums go through lanes by DPP instead of through LDS: at 567 rows
// 71 us a solve of 10 iterations instead of 115. Larger operators are read through
// one CU every iteration; small_solve_fits keeps them to what that costs less than
// the launches. The steps, decisions and tolerances are those of the launches in
// kernels.hip.
#include <hip/hip_runtime.h>

#include "ops.h"

namespace eqs {

constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int kSmallRows = 2;  // rows per thread at most
constexpr int kSmallLanes = 16;  // lanes of a coarse row

// Arrays copied to LDS: none, Q^T and B, or Q^T, B, Q and w.
enum Stage { kStageNone, kStageCoarse, kStageAll };

template <typename T>
struct SmallArgs {
    InstMap m;
    CsrView<T> Rt;       // Q_0^T
    SellView<T> Q;       // Q_0
    const T* B;          // the bottom's dense operator, n1 x n1
    const T* w;          // w D_0^-1
    int32_t n, n1;
    const double* rhs;
    double* x;
    double* mx_out;      // M x of the solution (may be NULL)
    double rtol;
    int32_t maxit, flexible, force;
    PcgScalars* host;
    PcgSummary* host_sum;
    int32_t rt_nnz, q_stored;
};

// Copies an array to LDS and returns where; at: the next free byte (16-aligned).
template <typename V>
__device__ __forceinline__ const V* small_copy(const V* src, int32_t count, char* lds, int32_t& at) {
    const int32_t bytes = count * (int32_t)sizeof(V), quads = bytes / 16;
    char* dst = lds + at;
#pragma unroll 4
    for (int32_t k = threadIdx.x; k < quads; k += kSmallThreads)
        reinterpret_cast<int4*>(dst)[k] = reinterpret_cast<const int4*>(src)[k];
    const int32_t k = quads * (16 / (int32_t)sizeof(V)) + (int32_t)threadIdx.x;  // fewer than 16 bytes are left
    if (k < count) reinterpret_cast<V*>(dst)[k] = src[k];
    at += (bytes + 15) & ~15;
    return reinterpret_cast<const V*>(dst);
}

// Sums of K values per thread over the workgroup, in a fixed order, for every
// thread. red: 2 x 3 x kSmallWaves doubles, used in halves by turns, so that one
// barrier per call is enough (the next use of a half is a barrier away).
template <int K>
__device__ __forceinline__ void small_sums(double (&v)[K], double* red, int& turn) {
    double* h = red + (turn & 1) * 3 * kSmallWaves;
    ++turn;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double t = wave_total(v[k]);
        if (lane == 63) h[k * kSmallWaves + wave] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double t[kSmallWaves];  // the same addresses for every lane: broadcasts
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) t[w] = h[k * kSmallWaves + w];
#pragma unroll
        for (int o = kSmallWaves / 2; o > 0; o >>= 1)
#pragma unroll
            for (int w = 0; w < o; ++w) t[w] += t[w + o];
        v[k] = t[0];
    }
}

// The values of a thread's rows of an operator: held in registers where that is
// cheap (by diagonals, one row of 7), else read at every product.
template <typename Op, int R>
struct SmallRows {
    __device__ __forceinline__ void load(const Op&, int, int32_t, const InstMap&) {}
    template <typename F>
    __device__ __forceinline__ auto sum(const Op& op, int, int64_t g, int32_t row, const InstMap& m, F f) const {
        return op.sum(g, row, m, 0, f);
    }
};
template <typename T>
struct SmallRows<DiaOp<T, 3>, 1> {
    T v[7];
    __device__ __forceinline__ void load(const DiaOp<T, 3>& op, int, int32_t row, const InstMap& m) {
        op.values(row, m, 0, v);
    }
    template <typename F>
    __device__ __forceinline__ T sum(const DiaOp<T, 3>& op, int, int64_t, int32_t row, const InstMap& m, F f) const {
        return op.product(row, m, 0, v, f);
    }
};

template <typename T, int R, int STAGE, typename OpM, typename OpA>
__global__ __launch_bounds__(kSmallThreads) void k_small_solve(SmallArgs<T> a, OpM M, OpA A) {
    extern __shared__ double lds[];
    double* rl = lds;                  // r
    double* zl = rl + a.n;             // z (the iterate while M x is formed)
    double* red = zl + a.n;            // 6 kSmallWaves
    T* b1 = reinterpret_cast<T*>(red + 6 * kSmallWaves);
    T* x1 = b1 + a.n1;
    const int tid = threadIdx.x;
    int turn = 0;
    CsrView<T> Rt = a.Rt;
    SellView<T> Q = a.Q;
    const T* B = a.B;
    const T* w = a.w;
    if (STAGE != kStageNone) {
        char* base = reinterpret_cast<char*>(lds);
        int32_t at = (int32_t)((reinterpret_cast<char*>(x1 + a.n1) - base + 15) & ~15);
        Rt.rp = small_copy(a.Rt.rp, a.n1 + 1, base, at);
        Rt.d16 = small_copy(a.Rt.d16, a.rt_nnz, base, at);
        Rt.val = small_copy(a.Rt.val, a.rt_nnz, base, at);
        B = small_copy(a.B, a.n1 * a.n1, base, at);
        if (STAGE == kStageAll) {
            Q.sptr = small_copy(a.Q.sptr, a.Q.n_slices + 1, base, at);
            Q.d16 = small_copy(a.Q.d16, a.q_stored, base, at);
            Q.val = small_copy(a.Q.val, a.q_stored, base, at);
            w = small_copy(a.w, a.n, base, at);
        }
    }
    // the rows of this thread in M's order; they own x, p, q and r's updates
    int32_t row[R];
    bool own[R];
    double x[R], p[R], q[R], f[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int64_t g = u * kSmallThreads + tid;
        own[u] = false;
        row[u] = 0;
        if (M.live(g)) {
            row[u] = M.row(g);
            own[u] = row[u] < a.n;
        }
        x[u] = own[u] ? a.x[row[u]] : 0.0;
        f[u] = own[u] ? a.rhs[row[u]] : 0.0;
        p[u] = q[u] = 0.0;
    }
    // and in Q's order, which form z
    int32_t rowz[R];
    SmallRows<OpM, R> mrows;
    SmallRows<OpA, R> arows;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int64_t g = u * kSmallThreads + tid;
        rowz[u] = g < (int64_t)a.Q.n_slices * 64 ? sell_perm_row<1>(a.Q.perm, g) : a.n;
        if (M.live(g)) mrows.load(M, u, row[u], a.m);
        if (rowz[u] < a.n) arows.load(A, u, rowz[u], a.m);
    }
    double bb = 0.0, rr = 0.0, tol2 = 0.0, relres = 0.0;
    // r = rhs - M x into rl; rr and bb
    auto residual = [&](bool store_mx) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (own[u]) zl[row[u]] = x[u];
        __syncthreads();
        double s[2] = {0.0, 0.0};
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int64_t g = u * kSmallThreads + tid;
            if (!M.live(g)) continue;
            const double mx = mrows.sum(M, u, g, row[u], a.m, [&](int32_t j) { return zl[j]; });
            if (!own[u]) continue;
            const double r = f[u] - mx;
            rl[row[u]] = r;
            if (store_mx && a.mx_out) a.mx_out[row[u]] = mx;
            s[0] += r * r;
            s[1] += f[u] * f[u];
        }
        small_sums(s, red, turn);
        rr = s[0];
        bb = s[1];
    };
    int32_t it = 0, done = 0, status = EQS_OK, restarts = 0, force = a.force;
    // the start's or the check's decision
    auto decide = [&](bool forced) {
        relres = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        done = 0;
        status = EQS_OK;
        if (bb == 0.0 || (rr <= tol2 && !forced)) {
            done = 1;
        } else if (!isfinite(rr) || !isfinite(bb)) {
            done = 1;
            status = EQS_ERR_BREAKDOWN;
        } else if (it >= a.maxit) {
            done = 1;
            status = EQS_ERR_NOT_CONVERGED;
        }
    };
    residual(false);
    tol2 = a.rtol * a.rtol * bb;
    decide(false);
    if (bb == 0.0)
#pragma unroll
        for (int u = 0; u < R; ++u) x[u] = 0.0;
    double rho = 0.0;
    for (;;) {
        bool fresh = true;
        while (!done) {
            // b_1 = Q^T r
            for (int32_t i0 = 0; i0 < a.n1; i0 += kSmallThreads / kSmallLanes) {
                const int32_t i = i0 + tid / kSmallLanes;
                if (i < a.n1) {  // whole lane groups leave together
                    const T v = csr_row<kSmallLanes>(Rt, i, tid % kSmallLanes, [&](int32_t j) { return (T)rl[j]; });
                    if (tid % kSmallLanes == 0) b1[i] = v;
                }
            }
            __syncthreads();
            // x_1 = B b_1
            for (int32_t i0 = 0; i0 < a.n1; i0 += kSmallThreads / kSmallLanes) {
                const int32_t i = i0 + tid / kSmallLanes;
                if (i < a.n1) {
                    const T* b = B + (int64_t)i * a.n1;
                    T acc = T(0);
                    for (int32_t k0 = tid % kSmallLanes; k0 < a.n1; k0 += 8 * kSmallLanes) {
                        T t[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) t[e] = b[min(k0 + e * kSmallLanes, a.n1 - 1)];
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int32_t k = k0 + e * kSmallLanes;
                            acc += k < a.n1 ? t[e] * b1[k] : T(0);
                        }
                    }
                    acc = group_sum<kSmallLanes>(acc);
                    if (tid % kSmallLanes == 0) x1[i] = acc;
                }
            }
            __syncthreads();
            // z = w (2 r - A w r) + Q x_1
            double s[2] = {0.0, 0.0};
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int64_t g = u * kSmallThreads + tid;
                if (g >= (int64_t)a.Q.n_slices * 64) continue;
                const int32_t i = rowz[u];
                const bool in = i < a.n;
                const double ri = in ? rl[i] : 0.0, zo = in ? zl[i] : 0.0;
                const T wi = in ? w[i] : T(0);
                const T qx = sell_accum<1>(Q, g, i, [&](int32_t j) { return x1[j]; });
                T ar = T(0);
                if (A.live(g)) {
                    if constexpr (OpA::kScaled) ar = arows.sum(A, u, g, i, a.m, [&](int32_t j) { return (T)rl[j]; });
                    else ar = arows.sum(A, u, g, i, a.m, [&](int32_t j) { return w[j] * (T)rl[j]; });
                }
                if (in) {
                    const T v = wi * (T(2) * (T)ri - ar) + qx;
                    zl[i] = (double)v;
                    s[0] += ri * (double)v;
                    s[1] += fresh ? 0.0 : ri * zo;
                }
            }
            small_sums(s, red, turn);
            if (!(s[0] > 0.0) || !isfinite(s[0])) {
                done = 1;
                status = EQS_ERR_BREAKDOWN;
                break;
            }
            const double beta = fresh ? 0.0 : (a.flexible ? (s[0] - s[1]) / rho : s[0] / rho);
            rho = s[0];
            // q = M z + beta q, p = z + beta p
            double d[1] = {0.0};
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int64_t g = u * kSmallThreads + tid;
                if (!M.live(g)) continue;
                const double mz = mrows.sum(M, u, g, row[u], a.m, [&](int32_t j) { return zl[j]; });
                if (!own[u]) continue;
                const double zi = zl[row[u]];
                p[u] = fresh ? zi : zi + beta * p[u];
                q[u] = fresh ? mz : mz + beta * q[u];
                d[0] += p[u] * q[u];
            }
            small_sums(d, red, turn);
            if (!(d[0] > 0.0) || !isfinite(d[0])) {
                done = 1;
                status = EQS_ERR_BREAKDOWN;
                break;
            }
            const double alpha = rho / d[0];
            double e[1] = {0.0};
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (own[u]) {
                    x[u] += alpha * p[u];
                    const double r = rl[row[u]] - alpha * q[u];
                    rl[row[u]] = r;
                    e[0] += r * r;
                }
            small_sums(e, red, turn);  // its barrier also publishes rl
            rr = e[0];
            relres = sqrt(rr / bb);
            ++it;
            fresh = false;
            if (rr <= tol2) {
                done = 1;
            } else if (!isfinite(rr)) {
                done = 1;
                status = EQS_ERR_BREAKDOWN;
            } else if (it >= a.maxit) {
                done = 1;
                status = EQS_ERR_NOT_CONVERGED;
            }
        }
        // the true residual; a solve that disagrees restarts from it
        residual(true);
        if (status != EQS_ERR_BREAKDOWN) decide(force != 0);
        force = 0;
        if (done || ++restarts > 4) break;
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (own[u]) a.x[row[u]] = x[u];
    if (tid == 0) {
        PcgScalars h{};
        h.bb = bb;
        h.rr = rr;
        h.rho = rho;
        h.tol2 = tol2;
        h.relres = relres;
        h.it = it;
        h.maxit = a.maxit;
        h.done = done;
        h.status = status;
        h.flexible = a.flexible;
        *a.host = h;
        PcgSummary v{};
        v.all_done = done;
        v.n_active = done ? 0 : 1;
        v.n_breakdown = status == EQS_ERR_BREAKDOWN;
        v.n_notconv = status == EQS_ERR_NOT_CONVERGED;
        v.n_zero_rhs = bb == 0.0;
        v.max_it = it;
        v.max_relres = isnan(relres) ? INFINITY : relres;
        *a.host_sum = v;
    }
}

constexpr size_t kSmallLds = 160 * 1024;  // of a CU
static size_t small_lds(const eqs_ctx* c, int64_t n, int64_t n1) {
    return sizeof(double) * (size_t)(2 * n + 6 * kSmallWaves) +
           (c->amg.precision == EQS_PREC_FP32 ? sizeof(float) : sizeof(double)) * (size_t)(2 * n1);
}

bool small_solve_fits(const eqs_ctx* c, int64_t n, int64_t nnz, int64_t n1, int64_t nnz_q) {
    const int64_t v = c->amg.precision == EQS_PREC_FP32 ? 4 : 8;
    const int64_t bytes = nnz * (8 + v + 4) + 2 * nnz_q * (v + 4) + n1 * n1 * v;  // read per iteration
    return c->small && n <= kSmallRows * kSmallThreads && small_lds(c, n, n1) <= 64 * 1024 && bytes <= kSmallBytes;
}

template <typename T>
static void launch(hipStream_t s, eqs_ctx* c, Hierarchy<T>& h, const double* rhs, double* x, int32_t maxit, double rtol,
                   double* mx_out) {
    Level<T>& l0 = h.lv[0];
    Level<T>& l1 = h.lv[1];
    const InstMap m{nullptr, nullptr, 1, (int32_t)c->n_free, 1, 1};
    const SmallArgs<T> a{m, cview(l0.R), view(l0.Q.sell), l1.dense_inv, l0.w, l0.n, l1.n, rhs, x, mx_out, rtol, maxit,
                         c->amg.flexible, c->test_reject_first ? 1 : 0, c->d_hscal, c->d_hsum, (int32_t)l0.R.nnz,
                         (int32_t)l0.Q.sell.stored};
    const int R = (l0.n + kSmallThreads - 1) / kSmallThreads;
    const auto pad = [](size_t b) { return (b + 15) & ~(size_t)15; };
    const size_t base = pad(small_lds(c, l0.n, l1.n));
    const size_t coarse = pad(4 * (size_t)(l1.n + 1)) + pad(2 * (size_t)a.rt_nnz) + pad(sizeof(T) * (size_t)a.rt_nnz) +
                          pad(sizeof(T) * (size_t)l1.n * l1.n);
    const size_t fine = pad(4 * (size_t)(l0.Q.sell.n_slices + 1)) + pad(2 * (size_t)a.q_stored) +
                        pad(sizeof(T) * (size_t)a.q_stored) + pad(sizeof(T) * (size_t)l0.n);
    const bool d16 = a.Rt.d16 && a.Q.d16 && !a.Q.pbase && !a.Rt.rbase;
    const int stage = !d16 ? kStageNone : base + coarse + fine <= kSmallLds ? kStageAll
                                      : base + coarse <= kSmallLds          ? kStageCoarse : kStageNone;
    const size_t lds = base + (stage != kStageNone ? coarse : 0) + (stage == kStageAll ? fine : 0);
    using OpT = double;
    EQS_WITH_OP(c->Mdia, view(c->M), {
        using OpM = std::decay_t<decltype(op)>;
        using OpA = typename OpM::template Of<T>;
        OpA oa;
        if constexpr (OpA::kScaled) oa = OpA{sview(l0)};
        else oa = dia_op<T, OpA::kDiagonals>(l0.D);
        const auto pick = [&](auto st) {
            constexpr int S = decltype(st)::value;
            return R == 1 ? k_small_solve<T, 1, S, OpM, OpA> : k_small_solve<T, 2, S, OpM, OpA>;
        };
        auto k = stage == kStageAll      ? pick(std::integral_constant<int, kStageAll>{})
                 : stage == kStageCoarse ? pick(std::integral_constant<int, kStageCoarse>{})
                                         : pick(std::integral_constant<int, kStageNone>{});
        hipLaunchKernelGGL(k, dim3(1), dim3(kSmallThreads), lds, s, a, op, oa);
    });
}

void small_solve(hipStream_t s, eqs_ctx* c, const double* rhs, double* x, int32_t maxit, double rtol, double* mx_out) {
    if (c->amg.precision == EQS_PREC_FP32) launch<float>(s, c, c->h32, rhs, x, maxit, rtol, mx_out);
    else launch<double>(s, c, c->h64, rhs, x, maxit, rtol, mx_out);
}

}  // namespace eqs
