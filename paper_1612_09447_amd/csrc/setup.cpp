// Host-side, once-per-context setup: input validation and node ordering,
// assembly of the constant permittivity matrix M on the free nodes (eq. (2)),
// the smoothed-aggregation AMG hierarchy that preconditions every M-solve
// (built once: Sec. II, the constant M turns the stage solves into a multiple
// right-hand-side problem), RKC coefficients (ref. [9] of the paper) and the
// upload of everything to device memory in SELL-64 form.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <numeric>

#include <functional>
#include <iterator>
#include <type_traits>

#include "eqs_internal.h"
#include "p2.h"

namespace eqs {

static constexpr double kEps0 = 8.8541878128e-12;  // F/m

// Edge vectors from p0 and their cross products: for a tet with edges
// e1, e2, e3 from p0, the rows of J^{-1} (J = [e1 e2 e3]) are
// (e2 x e3, e3 x e1, e1 x e2) / det with det = e1 . (e2 x e3); so the
// barycentric gradients are g_k = c_k / det and g_0 = -(g_1 + g_2 + g_3).
static double tet_cofactors(const double* p0, const double* p1, const double* p2, const double* p3,
                            double c[4][3]) {
    double e1[3], e2[3], e3[3];
    for (int d = 0; d < 3; ++d) {
        e1[d] = p1[d] - p0[d];
        e2[d] = p2[d] - p0[d];
        e3[d] = p3[d] - p0[d];
    }
    auto cross = [](const double* a, const double* b, double* o) {
        o[0] = a[1] * b[2] - a[2] * b[1];
        o[1] = a[2] * b[0] - a[0] * b[2];
        o[2] = a[0] * b[1] - a[1] * b[0];
    };
    cross(e2, e3, c[1]);
    cross(e3, e1, c[2]);
    cross(e1, e2, c[3]);
    for (int d = 0; d < 3; ++d) c[0][d] = -(c[1][d] + c[2][d] + c[3][d]);
    return e1[0] * c[1][0] + e1[1] * c[1][1] + e1[2] * c[1][2];
}

// ------------------------------------------------------------ validation
void validate_and_order(eqs_ctx* c) {
    const int64_t N = c->n_nodes;
    for (int64_t i = 0; i < 3 * N; ++i)
        if (!std::isfinite(c->xyz[i])) fail(EQS_ERR_NONFINITE, "non-finite node coordinate");
    const int npe = c->npe;
    for (int64_t e = 0; e < c->n_tets; ++e) {
        const int32_t* v = &c->tets[npe * e];
        for (int a = 0; a < npe; ++a)
            if (v[a] < 0 || v[a] >= N) fail(EQS_ERR_INVALID_ARG, "tet " + std::to_string(e) + " has a node id out of range");
        double cf[4][3];
        double det = tet_cofactors(&c->xyz[3 * (int64_t)v[0]], &c->xyz[3 * (int64_t)v[1]], &c->xyz[3 * (int64_t)v[2]],
                                   &c->xyz[3 * (int64_t)v[3]], cf);
        if (!(std::fabs(det) > 0) || !std::isfinite(det))
            fail(EQS_ERR_INVALID_ARG, "tet " + std::to_string(e) + " has zero volume");
    }
    std::vector<char> is_dir(N, 0);
    for (size_t k = 0; k < c->dir_nodes.size(); ++k) is_dir[c->dir_nodes[k]] = 1;
    c->n_dir = (int64_t)c->dir_nodes.size();
    c->n_free = N - c->n_dir;
    c->int_to_user.resize(N);
    int64_t f = 0, d = c->n_free;
    for (int64_t i = 0; i < N; ++i) {
        if (is_dir[i]) c->int_to_user[d++] = (int32_t)i;
        else c->int_to_user[f++] = (int32_t)i;
    }
    // instances: free rows of instance i are the free nodes of its node range,
    // contiguous because free nodes keep increasing user ids
    if (c->inst_node_off.empty()) {
        c->inst_node_off = {0, N};
        c->inst_tet_off = {0, c->n_tets};
    }
    c->n_inst = (int64_t)c->inst_node_off.size() - 1;
    c->inst_row_off.assign(c->n_inst + 1, 0);
    for (int64_t i = 0; i < c->n_inst; ++i) {
        int64_t nf = 0, nd = 0;
        for (int64_t v = c->inst_node_off[i]; v < c->inst_node_off[i + 1]; ++v) (is_dir[v] ? nd : nf)++;
        if (nd == 0) fail(EQS_ERR_INVALID_ARG, "instance " + std::to_string(i) + " has no Dirichlet node");
        if (nf == 0) fail(EQS_ERR_INVALID_ARG, "instance " + std::to_string(i) + " has no free node");
        if (c->n_inst > 1 && nf < 256)
            fail(EQS_ERR_INVALID_ARG, "instance " + std::to_string(i) + " has fewer than 256 free nodes");
        c->inst_row_off[i + 1] = c->inst_row_off[i] + (int32_t)nf;
    }
    for (int64_t i = 0; i < c->n_inst; ++i)
        for (int64_t e = c->inst_tet_off[i]; e < c->inst_tet_off[i + 1]; ++e)
            for (int a = 0; a < npe; ++a) {
                const int32_t v = c->tets[npe * e + a];
                if (v < c->inst_node_off[i] || v >= c->inst_node_off[i + 1])
                    fail(EQS_ERR_INVALID_ARG, "tet " + std::to_string(e) + " uses a node of another instance");
            }
    c->inst_iters.assign(c->n_inst, 0);
    c->inst_relres.assign(c->n_inst, 0.0);
}

// ----------------------------------------------------------- assembly of M
// Off-diagonal entries whose magnitude is at roundoff level against the
// diagonal, |a_ij| <= 1e-14 sqrt(a_ii a_jj), are dropped. On meshes built from
// right-angled (Kuhn) tets the P1 Laplacian has exact zeros on the face and
// body diagonals of every cube, i.e. about half of the structural entries.
static Csr<double> drop_zeros(const Csr<double>& A) {
    std::vector<double> d(A.n_rows, 0.0);
    for (int32_t i = 0; i < A.n_rows; ++i)
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (A.col[k] == i) d[i] = A.val[k];
    Csr<double> B;
    B.n_rows = A.n_rows;
    B.n_cols = A.n_cols;
    B.ptr.assign(A.n_rows + 1, 0);
    B.col.reserve(A.nnz());
    B.val.reserve(A.nnz());
    for (int32_t i = 0; i < A.n_rows; ++i) {
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) {
            const int32_t j = A.col[k];
            if (j != i && std::fabs(A.val[k]) <= 1e-14 * std::sqrt(std::fabs(d[i] * d[j]))) continue;
            B.col.push_back(j);
            B.val.push_back(A.val[k]);
        }
        B.ptr[i + 1] = (int32_t)B.col.size();
    }
    return B;
}

Csr<double> assemble_M_free(const eqs_ctx* c) {
    const int64_t N = c->n_nodes, T = c->n_tets, NF = c->n_free;
    std::vector<int32_t> u2i(N);
    for (int64_t i = 0; i < N; ++i) u2i[c->int_to_user[i]] = (int32_t)i;

    const int npe = c->npe;
    // node -> incident tets
    std::vector<int64_t> nt_ptr(N + 1, 0);
    for (int64_t e = 0; e < npe * T; ++e) nt_ptr[u2i[c->tets[e]] + 1]++;
    for (int64_t i = 0; i < N; ++i) nt_ptr[i + 1] += nt_ptr[i];
    std::vector<int32_t> nt(nt_ptr[N]);
    {
        std::vector<int64_t> fill(nt_ptr.begin(), nt_ptr.end() - 1);
        for (int64_t e = 0; e < T; ++e)
            for (int a = 0; a < npe; ++a) nt[fill[u2i[c->tets[npe * e + a]]]++] = (int32_t)e;
    }

    // row patterns: free neighbours through incident tets
    Csr<double> M;
    M.n_rows = M.n_cols = (int32_t)NF;
    M.ptr.assign(NF + 1, 0);
    std::vector<int32_t> buf;
    for (int pass = 0; pass < 2; ++pass) {
        int64_t pos = 0;
        for (int64_t i = 0; i < NF; ++i) {
            buf.clear();
            for (int64_t k = nt_ptr[i]; k < nt_ptr[i + 1]; ++k) {
                const int32_t* v = &c->tets[npe * (int64_t)nt[k]];
                for (int a = 0; a < npe; ++a) {
                    int32_t j = u2i[v[a]];
                    if (j < NF) buf.push_back(j);
                }
            }
            std::sort(buf.begin(), buf.end());
            buf.erase(std::unique(buf.begin(), buf.end()), buf.end());
            if (pass == 0) {
                pos += (int64_t)buf.size();
                if (pos > INT32_MAX) fail(EQS_ERR_INVALID_ARG, "M has more than 2^31 nonzeros");
                M.ptr[i + 1] = (int32_t)pos;
            } else {
                std::copy(buf.begin(), buf.end(), M.col.begin() + M.ptr[i]);
            }
        }
        if (pass == 0) {
            M.col.resize(M.ptr[NF]);
            M.val.assign(M.ptr[NF], 0.0);
        }
    }

    // values: P1 element matrices eps_e |T| g_a . g_b = eps_e c_a . c_b / (6 |det|);
    // second order: eps_e sum_q G_a(q) . G_b(q) / (24 |det|) (see p2.h)
    double A[kP2Nodes][kP2Nodes];
    for (int64_t e = 0; e < T; ++e) {
        const int32_t* vu = &c->tets[npe * e];
        int32_t v[kP2Nodes];
        for (int a = 0; a < npe; ++a) v[a] = u2i[vu[a]];
        double cf[4][3];
        double det = tet_cofactors(&c->xyz[3 * (int64_t)vu[0]], &c->xyz[3 * (int64_t)vu[1]], &c->xyz[3 * (int64_t)vu[2]],
                                   &c->xyz[3 * (int64_t)vu[3]], cf);
        const double eps = kEps0 * c->mats[c->tet_mat[e]].eps_r;
        if (npe == 4) {
            const double w = eps / (6.0 * std::fabs(det));
            for (int a = 0; a < 4; ++a)
                for (int b = 0; b < 4; ++b) A[a][b] = w * (cf[a][0] * cf[b][0] + cf[a][1] * cf[b][1] + cf[a][2] * cf[b][2]);
        } else {
            for (int a = 0; a < kP2Nodes; ++a)
                for (int b = 0; b < kP2Nodes; ++b) A[a][b] = 0.0;
            const double w = eps / (24.0 * std::fabs(det));
            for (int q = 0; q < 4; ++q) {
                double G[kP2Nodes][3];
                for (int a = 0; a < 4; ++a)
                    for (int d = 0; d < 3; ++d) G[a][d] = (4.0 * p2_lambda(q, a) - 1.0) * cf[a][d];
                for (int k = 0; k < 6; ++k) {
                    const int a = p2_edge_a(k), b = p2_edge_b(k);
                    for (int d = 0; d < 3; ++d) G[4 + k][d] = 4.0 * (p2_lambda(q, b) * cf[a][d] + p2_lambda(q, a) * cf[b][d]);
                }
                for (int a = 0; a < kP2Nodes; ++a)
                    for (int b = 0; b < kP2Nodes; ++b) A[a][b] += w * (G[a][0] * G[b][0] + G[a][1] * G[b][1] + G[a][2] * G[b][2]);
            }
        }
        for (int a = 0; a < npe; ++a) {
            if (v[a] >= NF) continue;
            const int32_t* cb = M.col.data() + M.ptr[v[a]];
            const int32_t* ce = M.col.data() + M.ptr[v[a] + 1];
            for (int b = 0; b < npe; ++b) {
                if (v[b] >= NF) continue;
                const int32_t* it = std::lower_bound(cb, ce, v[b]);
                M.val[it - M.col.data()] += A[a][b];
            }
        }
    }
    return drop_zeros(M);
}

// ------------------------------------------------------ sparse host algebra
static Csr<double> transpose(const Csr<double>& A) {
    Csr<double> T;
    T.n_rows = A.n_cols;
    T.n_cols = A.n_rows;
    T.ptr.assign(T.n_rows + 1, 0);
    for (int32_t k = 0; k < (int32_t)A.nnz(); ++k) T.ptr[A.col[k] + 1]++;
    for (int32_t i = 0; i < T.n_rows; ++i) T.ptr[i + 1] += T.ptr[i];
    T.col.resize(A.nnz());
    T.val.resize(A.nnz());
    std::vector<int32_t> fill(T.ptr.begin(), T.ptr.end() - 1);
    for (int32_t i = 0; i < A.n_rows; ++i)
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) {
            int32_t p = fill[A.col[k]]++;
            T.col[p] = i;
            T.val[p] = A.val[k];
        }
    return T;
}

// C = A B, row by row with a dense accumulator (columns sorted per row).
static Csr<double> spgemm(const Csr<double>& A, const Csr<double>& B) {
    Csr<double> C;
    C.n_rows = A.n_rows;
    C.n_cols = B.n_cols;
    C.ptr.assign(C.n_rows + 1, 0);
    std::vector<double> acc(B.n_cols, 0.0);
    std::vector<int32_t> mark(B.n_cols, -1), cols;
    for (int32_t i = 0; i < A.n_rows; ++i) {
        cols.clear();
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) {
            const int32_t r = A.col[k];
            const double a = A.val[k];
            for (int32_t m = B.ptr[r]; m < B.ptr[r + 1]; ++m) {
                const int32_t j = B.col[m];
                if (mark[j] != i) {
                    mark[j] = i;
                    acc[j] = 0.0;
                    cols.push_back(j);
                }
                acc[j] += a * B.val[m];
            }
        }
        std::sort(cols.begin(), cols.end());
        if ((int64_t)C.col.size() + (int64_t)cols.size() > INT32_MAX) fail(EQS_ERR_INVALID_ARG, "AMG product too large");
        for (int32_t j : cols) {
            C.col.push_back(j);
            C.val.push_back(acc[j]);
        }
        C.ptr[i + 1] = (int32_t)C.col.size();
    }
    return C;
}

static std::vector<double> diagonal(const Csr<double>& A) {
    std::vector<double> d(A.n_rows, 0.0);
    for (int32_t i = 0; i < A.n_rows; ++i)
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (A.col[k] == i) d[i] = A.val[k];
    return d;
}

// Spectral radius of D^{-1} A: power iteration (deterministic start), with a
// 5 % margin, capped by the Gershgorin bound max_i sum_j |a_ij| / a_ii.
static double spectral_radius_DinvA(const Csr<double>& A, const std::vector<double>& d) {
    const int32_t n = A.n_rows;
    double gersh = 0.0;
    for (int32_t i = 0; i < n; ++i) {
        double s = 0.0;
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) s += std::fabs(A.val[k]);
        gersh = std::max(gersh, s / d[i]);
    }
    std::vector<double> x(n), y(n);
    uint64_t st = 0x9E3779B97F4A7C15ull;
    for (int32_t i = 0; i < n; ++i) {
        st ^= st << 13; st ^= st >> 7; st ^= st << 17;
        x[i] = 0.5 + (double)(st >> 11) * (1.0 / 9007199254740992.0);
    }
    double lam = 0.0;
    for (int it = 0; it < 15; ++it) {
        double nx = 0.0, ny = 0.0;
        for (int32_t i = 0; i < n; ++i) {
            double s = 0.0;
            for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) s += A.val[k] * x[A.col[k]];
            y[i] = s / d[i];
            ny += y[i] * y[i];
            nx += x[i] * x[i];
        }
        lam = std::sqrt(ny / nx);
        double inv = 1.0 / std::sqrt(ny);
        for (int32_t i = 0; i < n; ++i) x[i] = y[i] * inv;
    }
    return std::min(gersh, 1.05 * lam);
}

// Greedy aggregation on the strength graph: (1) a node whose strong
// neighbours are all unassigned seeds an aggregate with them; (2) leftover
// nodes join the seeded aggregate they are most strongly tied to; (3) what is
// still unassigned forms aggregates with its unassigned strong neighbours.
static int32_t aggregate(const Csr<double>& A, const std::vector<double>& d, double theta,
                         std::vector<int32_t>& agg) {
    const int32_t n = A.n_rows;
    std::vector<char> strong(A.nnz(), 0);
    for (int32_t i = 0; i < n; ++i)
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) {
            int32_t j = A.col[k];
            if (j != i && std::fabs(A.val[k]) >= theta * std::sqrt(std::fabs(d[i] * d[j]))) strong[k] = 1;
        }
    agg.assign(n, -1);
    int32_t na = 0;
    for (int32_t i = 0; i < n; ++i) {
        if (agg[i] != -1) continue;
        bool free_nbhd = true, any = false;
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (strong[k]) {
                any = true;
                if (agg[A.col[k]] != -1) { free_nbhd = false; break; }
            }
        if (!any || !free_nbhd) continue;
        agg[i] = na;
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (strong[k]) agg[A.col[k]] = na;
        ++na;
    }
    std::vector<int32_t> seeded = agg;
    for (int32_t i = 0; i < n; ++i) {
        if (agg[i] != -1) continue;
        double best = -1.0;
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (strong[k] && seeded[A.col[k]] != -1 && std::fabs(A.val[k]) > best) {
                best = std::fabs(A.val[k]);
                agg[i] = seeded[A.col[k]];
            }
    }
    for (int32_t i = 0; i < n; ++i) {
        if (agg[i] != -1) continue;
        agg[i] = na;
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k)
            if (strong[k] && agg[A.col[k]] == -1) agg[A.col[k]] = na;
        ++na;
    }
    // number aggregates in the order of their first row, so coarse rows follow
    // fine rows (locality, and instances stay contiguous at every level)
    std::vector<int32_t> renum(na, -1);
    int32_t next = 0;
    for (int32_t i = 0; i < n; ++i)
        if (renum[agg[i]] < 0) renum[agg[i]] = next++;
    for (int32_t i = 0; i < n; ++i) agg[i] = renum[agg[i]];
    return na;
}

// Dense inverse of a small SPD matrix via Cholesky (column-major output).
static std::vector<double> dense_spd_inverse(const Csr<double>& A) {
    const int32_t n = A.n_rows;
    std::vector<double> L((size_t)n * n, 0.0);  // row-major lower factor
    for (int32_t i = 0; i < n; ++i)
        for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) L[(size_t)i * n + A.col[k]] = A.val[k];
    for (int32_t j = 0; j < n; ++j) {
        double s = L[(size_t)j * n + j];
        for (int32_t k = 0; k < j; ++k) s -= L[(size_t)j * n + k] * L[(size_t)j * n + k];
        if (!(s > 0)) fail(EQS_ERR_INVALID_ARG, "coarsest AMG matrix is not positive definite");
        const double ljj = std::sqrt(s);
        L[(size_t)j * n + j] = ljj;
        for (int32_t i = j + 1; i < n; ++i) {
            double t = L[(size_t)i * n + j];
            for (int32_t k = 0; k < j; ++k) t -= L[(size_t)i * n + k] * L[(size_t)j * n + k];
            L[(size_t)i * n + j] = t / ljj;
        }
    }
    std::vector<double> inv((size_t)n * n, 0.0), col(n);
    for (int32_t c = 0; c < n; ++c) {
        // solve L y = e_c, then L^T x = y
        for (int32_t i = 0; i < n; ++i) {
            double t = (i == c) ? 1.0 : 0.0;
            for (int32_t k = 0; k < i; ++k) t -= L[(size_t)i * n + k] * col[k];
            col[i] = t / L[(size_t)i * n + i];
        }
        for (int32_t i = n - 1; i >= 0; --i) {
            double t = col[i];
            for (int32_t k = i + 1; k < n; ++k) t -= L[(size_t)k * n + i] * col[k];
            col[i] = t / L[(size_t)i * n + i];
        }
        for (int32_t i = 0; i < n; ++i) inv[(size_t)c * n + i] = col[i];
    }
    return inv;
}

AmgHost build_sa_amg(const Csr<double>& M, const eqs_amg_params& p, bool keep_AP) {
    AmgHost h;
    Csr<double> A = M;
    for (;;) {
        const int32_t n = A.n_rows;
        const bool last = n <= p.coarse_max || (int32_t)h.A.size() + 1 >= p.max_levels;
        std::vector<double> d = diagonal(A);
        for (int32_t i = 0; i < n; ++i)
            if (!(d[i] > 0)) fail(EQS_ERR_INVALID_ARG, "matrix has a non-positive diagonal entry");
        if (last) {
            if (n > 4096) fail(EQS_ERR_INVALID_ARG, "AMG coarsening stalled above 4096 unknowns");
            h.coarse_inv = dense_spd_inverse(A);
            h.omega.push_back(0.0);
            h.A.push_back(std::move(A));
            break;
        }
        const double rho = spectral_radius_DinvA(A, d);
        std::vector<int32_t> agg;
        // strength threshold halves from level to level (Vanek, Mandel, Brezina 1996)
        const double theta_l = p.theta * std::ldexp(1.0, -(int)h.A.size());
        const int32_t nc = aggregate(A, d, theta_l, agg);
        if (nc >= n) fail(EQS_ERR_INVALID_ARG, "AMG aggregation did not coarsen");

        // tentative prolongator: column per aggregate, normalised
        std::vector<int32_t> size(nc, 0);
        for (int32_t i = 0; i < n; ++i) size[agg[i]]++;
        std::vector<double> w(nc);
        for (int32_t a = 0; a < nc; ++a) w[a] = 1.0 / std::sqrt((double)size[a]);

        // P = P_tent - (smooth_weight / rho) D^{-1} A P_tent
        const double sw = p.smooth_weight / rho;
        Csr<double> P;
        P.n_rows = n;
        P.n_cols = nc;
        P.ptr.assign(n + 1, 0);
        std::vector<int32_t> cols;
        std::vector<double> acc(nc, 0.0);
        std::vector<int32_t> mark(nc, -1);
        for (int32_t i = 0; i < n; ++i) {
            cols.clear();
            auto add = [&](int32_t a, double v) {
                if (mark[a] != i) { mark[a] = i; acc[a] = 0.0; cols.push_back(a); }
                acc[a] += v;
            };
            add(agg[i], w[agg[i]]);
            for (int32_t k = A.ptr[i]; k < A.ptr[i + 1]; ++k) {
                int32_t j = A.col[k];
                add(agg[j], -sw * A.val[k] / d[i] * w[agg[j]]);
            }
            std::sort(cols.begin(), cols.end());
            for (int32_t a : cols) {
                P.col.push_back(a);
                P.val.push_back(acc[a]);
            }
            P.ptr[i + 1] = (int32_t)P.col.size();
        }
        Csr<double> R = transpose(P);
        Csr<double> AP = spgemm(A, P);
        Csr<double> Ac = spgemm(R, AP);
        h.omega.push_back(p.jacobi_weight / rho);
        h.A.push_back(std::move(A));
        h.P.push_back(std::move(P));
        h.R.push_back(std::move(R));
        if (keep_AP) h.AP.push_back(std::move(AP));
        A = std::move(Ac);
    }
    return h;
}

// ---------------------------------------------------------------- RKC(s)
// Stability boundary beta(s) = (1 + w0) / w1 of RKC(s) (ref. [9]), damping 2/13.
double rkc_beta(int s) {
    const double w0 = 1.0 + (2.0 / 13.0) / ((double)s * s);
    double T0 = 1.0, T = w0, d0 = 0.0, d = 1.0, dd0 = 0.0, dd = 0.0;  // T_j, T_j', T_j'' at w0 (j = 1)
    for (int j = 2; j <= s; ++j) {
        const double Tn = 2.0 * w0 * T - T0, dn = 2.0 * T + 2.0 * w0 * d - d0, ddn = 4.0 * d + 2.0 * w0 * dd - dd0;
        T0 = T; T = Tn; d0 = d; d = dn; dd0 = dd; dd = ddn;
    }
    return (1.0 + w0) / (d / dd);
}

// Coefficients of the s-stage second-order RKC method (ref. [9]: Sommeijer,
// Shampine, Verwer), damping 2/13. Index j = 0..s; mu, nu, mut (mu~), gmt
// (gamma~) are used for j >= 2 (mut also for j = 1); c are the stage times.
void rkc_coefficients(int s, std::vector<double>& mu, std::vector<double>& nu, std::vector<double>& mut,
                      std::vector<double>& gmt, std::vector<double>& c) {
    const double w0 = 1.0 + (2.0 / 13.0) / ((double)s * s);
    std::vector<double> T(s + 1), T1(s + 1), T2(s + 1);  // Chebyshev T_j and derivatives at w0
    T[0] = 1.0; T1[0] = 0.0; T2[0] = 0.0;
    T[1] = w0;  T1[1] = 1.0; T2[1] = 0.0;
    for (int j = 2; j <= s; ++j) {
        T[j] = 2.0 * w0 * T[j - 1] - T[j - 2];
        T1[j] = 2.0 * T[j - 1] + 2.0 * w0 * T1[j - 1] - T1[j - 2];
        T2[j] = 4.0 * T1[j - 1] + 2.0 * w0 * T2[j - 1] - T2[j - 2];
    }
    const double w1 = T1[s] / T2[s];
    std::vector<double> b(s + 1), a(s + 1);
    for (int j = 2; j <= s; ++j) b[j] = T2[j] / (T1[j] * T1[j]);
    b[0] = b[1] = b[2];
    for (int j = 0; j <= s; ++j) a[j] = 1.0 - b[j] * T[j];
    mu.assign(s + 1, 0.0); nu.assign(s + 1, 0.0); mut.assign(s + 1, 0.0); gmt.assign(s + 1, 0.0); c.assign(s + 1, 0.0);
    mut[1] = b[1] * w1;
    c[1] = mut[1];
    for (int j = 2; j <= s; ++j) {
        mu[j] = 2.0 * b[j] * w0 / b[j - 1];
        nu[j] = -b[j] / b[j - 2];
        mut[j] = 2.0 * b[j] * w1 / b[j - 1];
        gmt[j] = -a[j - 1] * mut[j];
        c[j] = w1 * T2[j] / T1[j];
    }
}

// ------------------------------------------------------------------ upload
// Every device buffer of a context goes through dev_alloc: 256-byte granules,
// from hipMalloc or, when the caller gave a workspace, first fit from its free
// ranges.
static constexpr int64_t kGranule = 256;
static int64_t granules(size_t bytes) { return ((int64_t)std::max<size_t>(bytes, 1) + kGranule - 1) / kGranule * kGranule; }

static bool in_workspace(const eqs_ctx* c, const void* p) {
    return c->ws_base && (const char*)p >= c->ws_base && (const char*)p < c->ws_base + c->ws_size;
}

static void ws_reset(eqs_ctx* c) {
    c->ws_free.clear();
    c->ws_used = 0;
    if (c->ws_base && c->ws_size > 0) c->ws_free[0] = c->ws_size;
}

void* dev_alloc(eqs_ctx* c, size_t bytes) {
    const int64_t len = granules(bytes);
    void* p = nullptr;
    if (c->ws_base) {
        for (auto it = c->ws_free.begin(); it != c->ws_free.end(); ++it)
            if (it->second >= len) {
                const int64_t off = it->first, rest = it->second - len;
                c->ws_free.erase(it);
                if (rest > 0) c->ws_free[off + len] = rest;
                p = c->ws_base + off;
                break;
            }
        if (!p)
            fail(EQS_ERR_ALLOC, "workspace too small: " + std::to_string(len) + " more bytes needed with " +
                                    std::to_string(c->ws_size - c->ws_used) + " free (eqs_query gives the size)");
        c->ws_used += len;
    } else {
        hipError_t e = hipMalloc(&p, (size_t)len);
        if (e != hipSuccess) fail(EQS_ERR_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e));
        c->device_bytes += len;
    }
    c->allocations.push_back({p, (size_t)len});
    return p;
}

void dev_free(eqs_ctx* c, void* p) {
    if (!p) return;
    for (size_t k = 0; k < c->allocations.size(); ++k)
        if (c->allocations[k].first == p) {
            const int64_t len = (int64_t)c->allocations[k].second;
            if (in_workspace(c, p)) {
                // back to the free ranges, merged with its neighbours
                int64_t off = (char*)p - c->ws_base, n = len;
                auto nx = c->ws_free.lower_bound(off);
                if (nx != c->ws_free.end() && nx->first == off + n) {
                    n += nx->second;
                    nx = c->ws_free.erase(nx);
                }
                if (nx != c->ws_free.begin()) {
                    auto pv = std::prev(nx);
                    if (pv->first + pv->second == off) {
                        off = pv->first;
                        n += pv->second;
                        c->ws_free.erase(pv);
                    }
                }
                c->ws_free[off] = n;
                c->ws_used -= len;
            } else {
                (void)hipFree(p);
                c->device_bytes -= len;
            }
            c->allocations.erase(c->allocations.begin() + k);
            return;
        }
}

int64_t workspace_need(const eqs_ctx* c) {
    int64_t n = 0;
    for (const auto& a : c->allocations) n += (int64_t)a.second;
    return n + guess_pending_bytes(c);
}

template <typename T>
static void visit_sell(Sell<T>& S, const std::function<void(void**)>& f) {
    f((void**)&S.sptr);
    f((void**)&S.col);
    f((void**)&S.d16);
    f((void**)&S.pbase);
    f((void**)&S.val);
    f((void**)&S.perm);
}
template <typename T>
static void visit_spmat(SpMat<T>& A, const std::function<void(void**)>& f) {
    visit_sell(A.sell, f);
    f((void**)&A.rowptr);
    f((void**)&A.col);
    f((void**)&A.d16);
    f((void**)&A.rbase);
    f((void**)&A.val);
}
template <typename T>
static void visit_dia(Dia<T>& D, const std::function<void(void**)>& f) {
    f((void**)&D.val);
    f((void**)&D.offs);
}
template <typename T>
static void visit_hierarchy(Hierarchy<T>& h, const std::function<void(void**)>& f) {
    for (Level<T>& lv : h.lv) {
        visit_spmat(lv.A, f);
        visit_spmat(lv.P, f);
        visit_spmat(lv.R, f);
        visit_spmat(lv.GQ, f);
        visit_spmat(lv.Q, f);
        visit_dia(lv.D, f);
        f((void**)&lv.w);
        for (T** q : {&lv.dinv, &lv.sval, &lv.b, &lv.x, &lv.xs, &lv.res, &lv.dense_inv, &lv.coarse_R}) f((void**)q);
    }
}

void visit_device_ptrs(eqs_ctx* c, const std::function<void(void**)>& f) {
    f((void**)&c->d_tpack);
    f((void**)&c->d_kslots);
    f((void**)&c->d_kend);
    f((void**)&c->d_occ_off);
    f((void**)&c->d_occ);
    f((void**)&c->d_kx_part);
    f((void**)&c->d_bnodes);
    f((void**)&c->d_boff);
    f((void**)&c->d_cx);
    f((void**)&c->d_cy);
    f((void**)&c->d_cz);
    f((void**)&c->d_mats);
    f((void**)&c->d_ddrive);
    f((void**)&c->d_drives);
    f((void**)&c->d_int_to_user);
    visit_sell(c->M, f);
    visit_dia(c->Mdia, f);
    visit_hierarchy(c->h64, f);
    visit_hierarchy(c->h32, f);
    for (double** q : {&c->d_r, &c->d_z, &c->d_p, &c->d_q, &c->d_mx, &c->d_Y0, &c->d_Ya, &c->d_Yb, &c->d_Yc, &c->d_F0,
                       &c->d_F, &c->d_rhs, &c->d_rhs_alt, &c->d_tmpN, &c->d_tmpN2, &c->d_partials})
        f((void**)q);
    f((void**)&c->d_inst_row);
    f((void**)&c->d_blk_inst);
    f((void**)&c->d_scal);
    f((void**)&c->d_step);
    f((void**)&c->d_sum);
    f((void**)&c->d_force);
    GuessState& g = c->guess;
    for (double** q : {&g.d_S, &g.d_rprev, &g.d_alpha, &g.d_guard, &g.d_part}) f((void**)q);
    f((void**)&g.d_gstat);
    f((void**)&g.d_bx);
    f((void**)&g.d_bt);
    mlp_visit(g.net, f);
}

// Move every device buffer into [dev, dev + bytes) (dev NULL: into buffers
// the library allocates), packed in allocation order, and remap every pointer
// that points into an old buffer (interior pointers keep their offset). A
// buffer that no visited pointer reaches stops the move before anything
// changes.
void set_workspace(eqs_ctx* c, void* dev, int64_t bytes) {
    EQS_HIP(hipStreamSynchronize(c->stream));
    if (c->guess.tstream) EQS_HIP(hipStreamSynchronize(c->guess.tstream));
    const std::vector<std::pair<void*, size_t>> old = c->allocations;
    auto owner = [&](const void* p) -> int {
        for (size_t k = 0; k < old.size(); ++k)
            if ((const char*)p >= (const char*)old[k].first && (const char*)p < (const char*)old[k].first + old[k].second)
                return (int)k;
        return -1;
    };
    std::vector<int> hits(old.size(), 0);
    visit_device_ptrs(c, [&](void** pp) {
        if (*pp) {
            const int k = owner(*pp);
            if (k >= 0) hits[k]++;
        }
    });
    for (size_t k = 0; k < old.size(); ++k)
        if (!hits[k]) fail(EQS_ERR_STATE, "internal: a device buffer of the context is not reachable for the move");
    int64_t total = 0;
    for (const auto& a : old) total += (int64_t)a.second;
    if (dev) {
        if (bytes < total)
            fail(EQS_ERR_INVALID_ARG, "workspace too small: " + std::to_string(total) + " bytes needed, " +
                                          std::to_string(bytes) + " given");
        for (const auto& a : old)
            if ((const char*)a.first < (const char*)dev + bytes && (const char*)dev < (const char*)a.first + a.second)
                fail(EQS_ERR_INVALID_ARG, "workspace overlaps the context's own device memory");
    }
    std::vector<void*> fresh(old.size(), nullptr);
    int64_t off = 0;
    try {
        for (size_t k = 0; k < old.size(); ++k) {
            if (dev) {
                fresh[k] = (char*)dev + off;
                off += (int64_t)old[k].second;
            } else {
                hipError_t e = hipMalloc(&fresh[k], old[k].second);
                if (e != hipSuccess) fail(EQS_ERR_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e));
            }
        }
        for (size_t k = 0; k < old.size(); ++k)
            EQS_HIP(hipMemcpyAsync(fresh[k], old[k].first, old[k].second, hipMemcpyDeviceToDevice, c->stream));
        EQS_HIP(hipStreamSynchronize(c->stream));
    } catch (...) {
        if (!dev)
            for (void* p : fresh)
                if (p) (void)hipFree(p);
        throw;
    }
    release_graphs(c);  // captured iterations hold the old addresses
    visit_device_ptrs(c, [&](void** pp) {
        if (!*pp) return;
        const int k = owner(*pp);
        if (k >= 0) *pp = (char*)fresh[k] + ((char*)*pp - (char*)old[k].first);
    });
    for (size_t k = 0; k < old.size(); ++k)
        if (!in_workspace(c, old[k].first)) (void)hipFree(old[k].first);
    c->allocations.clear();
    for (size_t k = 0; k < old.size(); ++k) c->allocations.push_back({fresh[k], old[k].second});
    c->ws_base = (char*)dev;
    c->ws_size = dev ? bytes : 0;
    c->ws_free.clear();
    c->ws_used = dev ? total : 0;
    if (dev && bytes > total) c->ws_free[total] = bytes - total;
    c->device_bytes = dev ? 0 : total;
}

template <typename T>
static T* upload_vec(eqs_ctx* c, const std::vector<T>& v) {
    T* d = (T*)dev_alloc(c, v.size() * sizeof(T));
    if (!v.empty()) EQS_HIP(hipMemcpy(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    return d;
}

template <typename T>
Sell<T> to_sell(eqs_ctx* c, const Csr<double>& A, int lanes, bool sorted, const Csr<double>* key, int32_t split) {
    if (lanes != 1 && lanes != 2 && lanes != 4 && lanes != 8) fail(EQS_ERR_STATE, "SELL lanes per row must be 1, 2, 4 or 8");
    const int32_t rows_per = kSlice / lanes;  // rows of one slice
    const int32_t window = 4 * rows_per;      // rows of one 256-thread window
    Sell<T> S;
    S.n_rows = A.n_rows;
    S.n_cols = A.n_cols;
    S.lanes = lanes;
    S.n_slices = (A.n_rows + rows_per - 1) / rows_per;
    // pos2row[k]: the row stored at position k (positions past n_rows are
    // phantom rows >= n_rows); sorted: longest rows first within each window
    const int32_t n_pos = S.n_slices * rows_per;
    std::vector<int32_t> pos2row((size_t)n_pos);
    for (int32_t k = 0; k < n_pos; ++k) pos2row[(size_t)k] = k;
    auto len = [&](int32_t r) { return r < A.n_rows ? A.ptr[r + 1] - A.ptr[r] : 0; };
    auto key_len = [&](int32_t r) { return !key ? len(r) : r < A.n_rows ? key->ptr[r + 1] - key->ptr[r] : 0; };
    if (sorted)
        for (int32_t w0 = 0; w0 < n_pos; w0 += window) {
            const int32_t w1 = std::min(n_pos, w0 + window);
            std::stable_sort(pos2row.begin() + w0, pos2row.begin() + w1,
                             [&](int32_t a, int32_t b) { return key_len(a) > key_len(b); });
        }
    // lane l of slice s serves the row at position s * rows_per + l / lanes and
    // holds the row's entries l % lanes + lanes * k, k = 0 .. w-1; columns from
    // `at_col` on begin at a pair of their own in all rows of a slice
    std::vector<int32_t> sptr, col;
    std::vector<T> val;
    auto lay_out = [&](int32_t at_col) {
        auto first_len = [&](int32_t r) {  // entries before at_col
            if (r >= A.n_rows) return 0;
            if (at_col >= A.n_cols) return len(r);
            return (int32_t)(std::lower_bound(A.col.begin() + A.ptr[r], A.col.begin() + A.ptr[r + 1], at_col) -
                             (A.col.begin() + A.ptr[r]));
        };
        auto lane_pairs = [&](int32_t n) { return ((n + lanes - 1) / lanes + 1) / 2; };
        sptr.assign(S.n_slices + 1, 0);
        std::vector<int32_t> w1((size_t)S.n_slices, 0);  // pairs before at_col
        for (int32_t s = 0; s < S.n_slices; ++s) {
            int32_t p1 = 0, p2 = 0;
            for (int32_t k = s * rows_per; k < (s + 1) * rows_per; ++k) {
                const int32_t n1 = first_len(pos2row[k]);
                p1 = std::max(p1, lane_pairs(n1));
                p2 = std::max(p2, lane_pairs(len(pos2row[k]) - n1));
            }
            w1[(size_t)s] = p1;
            const int64_t next = (int64_t)sptr[s] + (int64_t)(p1 + p2) * 2 * kSlice;
            if (next > INT32_MAX) fail(EQS_ERR_INVALID_ARG, "matrix too large for SELL offsets");
            sptr[s + 1] = (int32_t)next;
        }
        S.stored = sptr[S.n_slices];
        col.assign(S.stored, 0);
        val.assign(S.stored, T(0));
        for (int32_t s = 0; s < S.n_slices; ++s) {
            const int32_t w = (sptr[s + 1] - sptr[s]) / kSlice, wa = 2 * w1[(size_t)s];
            for (int32_t l = 0; l < kSlice; ++l) {
                const int32_t r = pos2row[(size_t)(s * rows_per + l / lanes)], part = l % lanes;
                const int32_t n = len(r), n1 = first_len(r);
                for (int32_t k = 0; k < w; ++k) {
                    const int64_t at = sptr[s] + (int64_t)(k >> 1) * 2 * kSlice + 2 * l + (k & 1);
                    const bool one = k < wa;
                    const int32_t e = one ? k * lanes + part : n1 + (k - wa) * lanes + part, end = one ? n1 : n;
                    if (e < end) {
                        col[at] = A.col[A.ptr[r] + e];
                        val[at] = (T)A.val[A.ptr[r] + e];
                    } else {  // the part's last column, or the row's
                        col[at] = end > (one ? 0 : n1) ? A.col[A.ptr[r] + end - 1] : n > 0 ? A.col[A.ptr[r] + n - 1] : 0;
                    }
                }
            }
        }
    };
    lay_out(A.n_cols);
    // 16-bit offsets from offset_base(row) when every stored column allows
    // (padding of rows past n_rows points at the last column)
    bool fits = c->index16 && A.n_cols > 0;
    std::vector<int16_t> d16;
    if (fits) {
        d16.assign(S.stored, 0);
        for (int32_t s = 0; s < S.n_slices && fits; ++s) {
            const int32_t w = (sptr[s + 1] - sptr[s]) / kSlice;
            for (int32_t l = 0; l < kSlice && fits; ++l) {
                const int32_t r = pos2row[(size_t)(s * rows_per + l / lanes)];
                const int64_t base = offset_base(r, A.n_rows, A.n_cols);
                for (int32_t k = 0; k < w; ++k) {
                    const int64_t at = sptr[s] + (int64_t)(k >> 1) * 2 * kSlice + 2 * l + (k & 1);
                    const int64_t d = (r < A.n_rows ? (int64_t)col[at] : (int64_t)A.n_cols - 1) - base;
                    if (d < -32767 || d > 32767) {
                        fits = false;
                        break;
                    }
                    d16[at] = (int16_t)d;
                }
            }
        }
    }
    // else from a base of each pair of entries (of one slice), when no 128 columns
    // of a pair span more than 65535
    std::vector<int32_t> pbase;
    auto by_pairs = [&]() {
        const int64_t np = S.stored / (2 * kSlice);
        pbase.assign((size_t)np, 0);
        d16.resize((size_t)S.stored);
        for (int32_t s = 0; s < S.n_slices; ++s) {
            // lanes of rows that are there: their padding keeps the row's own column (0 times
            // another row's operand is not 0 where that is no number)
            const int32_t rows = std::min(rows_per, (int32_t)std::max(0, A.n_rows - s * rows_per));
            const bool whole = rows == rows_per;
            for (int64_t q = sptr[s] / (2 * kSlice); q < sptr[s + 1] / (2 * kSlice); ++q) {
                const int32_t* p = &col[(size_t)q * 2 * kSlice];
                int32_t lo = INT32_MAX, hi = 0;
                for (int e = 0; e < 2 * kSlice; ++e)
                    if (whole || pos2row[(size_t)(s * rows_per + (e / 2) / lanes)] < A.n_rows) {
                        lo = std::min(lo, p[e]);
                        hi = std::max(hi, p[e]);
                    }
                if (hi - lo > 65535) return false;
                pbase[(size_t)q] = lo + 32768;
                for (int e = 0; e < 2 * kSlice; ++e)
                    d16[(size_t)q * 2 * kSlice + e] = (int16_t)(std::min(std::max(p[e], lo), hi) - lo - 32768);
            }
        }
        return true;
    };
    if (!fits && c->index16 && A.n_cols > 0) {
        fits = by_pairs();
        if (!fits && split > 0 && split < A.n_cols) {
            lay_out(split);
            fits = by_pairs();
            if (!fits) lay_out(A.n_cols);
        }
        if (fits) S.pbase = upload_vec(c, pbase);
    }
    S.sptr = upload_vec(c, sptr);
    if (fits) S.d16 = upload_vec(c, d16);
    else S.col = upload_vec(c, col);
    S.val = upload_vec(c, val);
    if (sorted) {
        std::vector<uint8_t> perm((size_t)n_pos);
        for (int32_t k = 0; k < n_pos; ++k) perm[(size_t)k] = (uint8_t)(pos2row[(size_t)k] - (k / window) * window);
        S.perm = upload_vec(c, perm);
    }
    return S;
}

template Sell<double> to_sell<double>(eqs_ctx*, const Csr<double>&, int, bool, const Csr<double>*, int32_t);
template Sell<float> to_sell<float>(eqs_ctx*, const Csr<double>&, int, bool, const Csr<double>*, int32_t);

// CSR column ids: 16-bit offsets from offset_base(row) when every entry
// allows, else from a base of the row's own, else absolute.
template <typename T>
static void upload_csr_cols(eqs_ctx* c, SpMat<T>& S, const Csr<double>& A) {
    bool fits = c->index16 && A.n_cols > 0;
    std::vector<int16_t> d16;
    if (fits) {
        d16.resize(A.col.size());
        for (int32_t r = 0; r < A.n_rows && fits; ++r) {
            const int64_t base = offset_base(r, A.n_rows, A.n_cols);
            for (int32_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
                const int64_t d = (int64_t)A.col[k] - base;
                if (d < -32767 || d > 32767) {
                    fits = false;
                    break;
                }
                d16[k] = (int16_t)d;
            }
        }
    }
    if (!fits && c->index16 && A.n_cols > 0) {  // from a base of each row, where no row spans more than 65535
        std::vector<int32_t> rbase((size_t)A.n_rows, 0);
        fits = true;
        for (int32_t r = 0; r < A.n_rows && fits; ++r) {
            if (A.ptr[r] == A.ptr[r + 1]) continue;
            const auto mm = std::minmax_element(A.col.begin() + A.ptr[r], A.col.begin() + A.ptr[r + 1]);
            fits = *mm.second - *mm.first <= 65535;
            rbase[(size_t)r] = *mm.first + 32768;
            for (int32_t k = A.ptr[r]; k < A.ptr[r + 1] && fits; ++k) d16[(size_t)k] = (int16_t)(A.col[k] - rbase[(size_t)r]);
        }
        if (fits) S.rbase = upload_vec(c, rbase);
    }
    if (fits) S.d16 = upload_vec(c, d16);
    else S.col = upload_vec(c, A.col);
}

// Layout choice: rows of up to 16 entries go one lane per row (SELL-64);
// longer rows get L = 2^ceil(log2(mean/2)) lanes (2 <= L <= 64), so each lane
// sums about two entries per pass and a wavefront covers 64/L rows.
// Whether storing the rows of a one-lane-per-row SELL operator longest first
// within each 256-row window (a row order) pays: when it saves a tenth of the
// stored entries. Rows of different lengths that alternate (the vertex and
// edge nodes of second-order tets: 1.57 stored entries per nonzero in the
// natural order, 1.10 sorted) gain; the nearly uniform rows of first-order
// tets (1.01) do not.
static bool row_order_pays(const Csr<double>& A) {
    const int32_t n = A.n_rows;
    if (n <= 0) return false;
    auto len = [&](int32_t r) { return r < n ? A.ptr[r + 1] - A.ptr[r] : 0; };
    const int32_t n_pos = ((n + kSlice - 1) / kSlice) * kSlice;
    int64_t plain = 0, sorted = 0;
    std::vector<int32_t> w;
    for (int32_t w0 = 0; w0 < n_pos; w0 += 4 * kSlice) {
        const int32_t w1 = std::min(n_pos, w0 + 4 * kSlice);
        w.clear();
        for (int32_t r = w0; r < w1; ++r) w.push_back(len(r));
        for (int32_t s0 = 0; s0 < (int32_t)w.size(); s0 += kSlice)
            plain += (int64_t)kSlice * *std::max_element(w.begin() + s0, w.begin() + std::min((int32_t)w.size(), s0 + kSlice));
        std::sort(w.begin(), w.end(), std::greater<int32_t>());
        for (int32_t s0 = 0; s0 < (int32_t)w.size(); s0 += kSlice) sorted += (int64_t)kSlice * w[(size_t)s0];
    }
    return sorted * 10 <= plain * 9;
}

// The upper diagonals (offsets, per instance) of a symmetric matrix that has at
// most kMaxDiagonals of them per instance; 3 or 7 are stored (the 7-point and
// 15-point stencils of structured numberings), with at most half as many zeros
// as entries in them. Empty: not such a matrix. Meshes numbered along their axes
// give few diagonals whatever their geometry; others do not.
static std::vector<std::vector<int32_t>> diagonals_of(const eqs_ctx* c, const Csr<double>& A, int& K) {
    std::vector<std::vector<int32_t>> off((size_t)c->n_inst);
    K = 0;
    int64_t upper = 0;
    for (int64_t i = 0; i < c->n_inst; ++i) {
        std::vector<int32_t>& o = off[(size_t)i];
        for (int32_t r = c->inst_row_off[i]; r < c->inst_row_off[i + 1]; ++r) {
            bool diag = false;
            for (int32_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
                const int32_t d = A.col[k] - r;
                if (d == 0) diag = true;
                if (d <= 0) continue;
                ++upper;
                auto it = std::lower_bound(o.begin(), o.end(), d);
                if (it == o.end() || *it != d) {
                    if (o.size() == (size_t)kMaxDiagonals) return {};
                    o.insert(it, d);
                }
            }
            if (!diag) return {};
        }
        K = std::max(K, (int)o.size());
    }
    K = K <= 3 ? 3 : kMaxDiagonals;
    if (2 * ((int64_t)K * A.n_rows - upper) > upper) return {};
    for (auto& o : off)  // unused diagonals hold zeros only; offset 0 reads the row itself
        o.resize((size_t)K, 0);
    return off;
}

// By diagonals, or K = 0 where that does not apply (diagonals_of) or the stored
// triangles are not equal bit for bit.
template <typename T>
static Dia<T> to_dia(eqs_ctx* c, const Csr<double>& A) {
    Dia<T> D;
    if (!c->diagonals || A.n_rows != A.n_cols || A.n_rows == 0) return D;
    int K = 0;
    const auto off = diagonals_of(c, A, K);
    if (off.empty()) return D;
    const int64_t n = A.n_rows;
    std::vector<double> val((size_t)((K + 1) * n), 0.0);
    for (int64_t i = 0; i < c->n_inst; ++i) {
        const std::vector<int32_t>& o = off[(size_t)i];
        auto which = [&](int32_t d) {
            int k = 0;
            while (o[(size_t)k] != d) ++k;
            return k;
        };
        for (int32_t r = c->inst_row_off[i]; r < c->inst_row_off[i + 1]; ++r)
            for (int32_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
                const int32_t d = A.col[k] - r;
                if (d >= 0) val[(size_t)((d == 0 ? 0 : which(d) + 1) * n + r)] = A.val[k];
            }
        for (int32_t r = c->inst_row_off[i]; r < c->inst_row_off[i + 1]; ++r)
            for (int32_t k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
                const int32_t d = r - A.col[k];
                if (d <= 0) continue;
                int q = 0;  // a lower offset without an upper entry: not symmetric
                while (q < K && o[(size_t)q] != d) ++q;
                if (q == K || val[(size_t)((q + 1) * n + A.col[k])] != A.val[k]) return D;
            }
    }
    D.K = K;
    D.n = (int32_t)n;
    for (int k = 0; k < K; ++k) D.off[k] = off[0][(size_t)k];
    if (c->n_inst > 1) {
        std::vector<int32_t> all;
        for (const auto& o : off) all.insert(all.end(), o.begin(), o.end());
        D.offs = upload_vec(c, all);
    }
    D.val = upload_vec(c, std::vector<T>(val.begin(), val.end()));
    return D;
}

template <typename T>
SpMat<T> to_spmat(eqs_ctx* c, const Csr<double>& A) {
    SpMat<T> S;
    S.n_rows = A.n_rows;
    S.n_cols = A.n_cols;
    S.nnz = A.nnz();
    const double mean = A.n_rows ? (double)A.nnz() / A.n_rows : 0.0;
    if (mean <= 16.0) {
        S.fmt = FMT_SELL;
        S.sell = to_sell<T>(c, A, 1);
        return S;
    }
    S.fmt = FMT_CSR;
    int L = 2;
    while (L < 64 && L < mean / 2.0) L *= 2;
    S.lanes = L;
    std::vector<T> v(A.val.size());
    for (size_t k = 0; k < v.size(); ++k) v[k] = (T)A.val[k];
    S.rowptr = upload_vec(c, A.ptr);
    upload_csr_cols(c, S, A);
    S.val = upload_vec(c, v);
    return S;
}
template SpMat<double> to_spmat<double>(eqs_ctx*, const Csr<double>&);
template SpMat<float> to_spmat<float>(eqs_ctx*, const Csr<double>&);

template <typename T>
static void free_spmat(eqs_ctx* c, SpMat<T>& S) {
    dev_free(c, S.sell.sptr);
    dev_free(c, S.sell.col);
    dev_free(c, S.sell.d16);
    dev_free(c, S.sell.pbase);
    dev_free(c, S.sell.val);
    dev_free(c, S.sell.perm);
    dev_free(c, S.rowptr);
    dev_free(c, S.col);
    dev_free(c, S.d16);
    dev_free(c, S.rbase);
    dev_free(c, S.val);
    S = SpMat<T>{};
}

// Autotuner: upload the operator in every candidate layout (SELL with 1 lane
// per row, and with 2, 4, 8 while each lane keeps 1.5 entries or more, each
// also with rows sorted by length within 256-thread windows (the products and
// the smoothers write only rows of their own window);
// CSR with L = 2..64 lanes per row up to about twice the mean row length, and
// with one lane per row for rows of up to 8 entries on average), time y = A x
// with HIP events on the context's stream (median of 5 rounds of 8 back-to-back launches, after a warm-up round) and
// keep the fastest.
template <typename T>
static SpMat<T> tuned_spmat(eqs_ctx* c, const Csr<double>& A, const char* what, bool sell_only = false,
                             bool allow_sorted = false, int32_t split = 0) {
    if (sell_only) {  // the finest operator: its post-smoothing kernel writes per-block CG partials
        SpMat<T> S;
        S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
        S.fmt = FMT_SELL;
        S.sell = to_sell<T>(c, A, 1, row_order_pays(A));
        S.sell.xcd = 1;  // the finest smoothers walk their row blocks in the XCD order (row_block in sell.h)
        c->tune_log += std::string(what) + ": sell64" + (S.sell.perm ? "s" : "") + " (finest level), " +
                       (S.sell.d16 ? "16-bit column offsets\n" : "32-bit columns\n");
        return S;
    }
    if (c->force_layout >= 0) {
        SpMat<T> S;
        if (c->force_layout == 0) {
            S = to_spmat<T>(c, A);
            if (S.fmt == FMT_SELL) {  // short rows: CSR with 2 lanes
                free_spmat(c, S);
                S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
                S.fmt = FMT_CSR;
                S.lanes = 2;
                std::vector<T> v(A.val.size());
                for (size_t k = 0; k < v.size(); ++k) v[k] = (T)A.val[k];
                S.rowptr = upload_vec(c, A.ptr);
                upload_csr_cols(c, S, A);
                S.val = upload_vec(c, v);
            }
        } else {
            S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
            S.fmt = FMT_SELL;
            S.sell = to_sell<T>(c, A, c->force_layout, c->force_sorted && allow_sorted, nullptr, split);
            S.sell.unroll = c->force_unroll;
        }
        c->tune_log += std::string(what) + ": layout set by EQS_LAYOUT\n";
        return S;
    }
    if (!c->autotune || A.n_rows == 0) return to_spmat<T>(c, A);
    const double mean = (double)A.nnz() / A.n_rows;
    auto make_csr = [&](int L) {
        SpMat<T> S;
        S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
        S.fmt = FMT_CSR;
        S.lanes = L;
        std::vector<T> v(A.val.size());
        for (size_t k = 0; k < v.size(); ++k) v[k] = (T)A.val[k];
        S.rowptr = upload_vec(c, A.ptr);
        upload_csr_cols(c, S, A);
        S.val = upload_vec(c, v);
        return S;
    };
    const std::string key = std::string(what) + " " + std::to_string(A.n_rows) + "x" + std::to_string(A.n_cols) + " " +
                            std::to_string(A.nnz());
    {
        auto it = c->tune_replay.find(key);
        if (it != c->tune_replay.end()) {  // a recorded choice: rebuild it without timing
            char kind[8] = {0};
            int L = 0, sorted = 0, U = 8;
            const int n = std::sscanf(it->second.c_str(), "%7s %d %d %d", kind, &L, &sorted, &U);
            SpMat<T> S;
            if (n >= 2 && std::string(kind) == "csr" && L >= 1 && L <= 64 && (L & (L - 1)) == 0) {
                S = make_csr(L);
            } else if (n == 4 && std::string(kind) == "sell" && (L == 1 || L == 2 || L == 4 || L == 8) &&
                       (U == 4 || U == 8 || U == 16)) {
                S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
                S.fmt = FMT_SELL;
                S.sell = to_sell<T>(c, A, L, sorted != 0 && allow_sorted, nullptr, split);
                S.sell.unroll = U;
            } else {
                fail(EQS_ERR_INVALID_ARG, "tuning record: bad entry for " + key + ": " + it->second);
            }
            c->tune_log += key + " -> " + it->second + " (tuning record)\n";
            return S;
        }
    }
    T* x = (T*)dev_alloc(c, sizeof(T) * std::max<int32_t>(A.n_cols, 1));
    T* y = (T*)dev_alloc(c, sizeof(T) * std::max<int32_t>(A.n_rows, 1));
    {
        std::vector<T> ones(std::max<int32_t>(A.n_cols, 1), T(1));
        EQS_HIP(hipMemcpy(x, ones.data(), sizeof(T) * ones.size(), hipMemcpyHostToDevice));
    }
    SpMat<T> best;
    double best_ms = 1e300;
    std::string best_name;
    std::string tried;
    auto consider = [&](SpMat<T> cand, const std::string& name) {
        const double ms = time_mv<T>(c, cand, x, y, 5);
        if (c->tune_verbose) {
            char t[96];
            std::snprintf(t, sizeof t, " %s %.1f", name.c_str(), ms * 1e3);
            tried += t;
        }
        if (ms < best_ms) {
            if (best.n_rows || best.nnz) free_spmat(c, best);
            best = cand;
            best_ms = ms;
            best_name = name;
        } else {
            free_spmat(c, cand);
        }
    };
    for (int L = 1; L <= 8; L *= 2) {
        if (L > 1 && mean < 1.5 * L) break;  // lanes with about one entry or less
        for (int sorted = 0; sorted <= (allow_sorted ? 1 : 0); ++sorted) {
            SpMat<T> S;
            S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
            S.fmt = FMT_SELL;
            S.sell = to_sell<T>(c, A, L, sorted != 0, nullptr, split);
            // the group size, timed on the product (the coarse smoothing kernels
            // take the same; the finest level's keep 8)
            {
                const double per_lane = mean / L;
                double best_u_ms = 1e300;
                int best_u = 8;
                for (int U : {4, 8, 16}) {
                    if (U == 16 && per_lane < 6.0) continue;
                    S.sell.unroll = U;
                    const double ms = time_mv<T>(c, S, x, y, 5);
                    if (c->tune_verbose) {
                        char t[64];
                        std::snprintf(t, sizeof t, " [u%d %.1f]", U, ms * 1e3);
                        tried += t;
                    }
                    if (ms < best_u_ms) {
                        best_u_ms = ms;
                        best_u = U;
                    }
                }
                S.sell.unroll = best_u;
            }
            consider(S, std::string("sell64") + (L > 1 ? "x" + std::to_string(L) : "") + (sorted ? "s" : "") +
                            (S.sell.pbase ? "/p16" : S.sell.d16 ? "/i16" : "") + (S.sell.unroll != 8 ? "/u" + std::to_string(S.sell.unroll) : ""));
        }
    }
    for (int L = (mean <= 8.0 ? 1 : 2); L <= 64; L *= 2) {
        if (L > 2 && L / 2 > 2.0 * mean) break;
        SpMat<T> S;
        S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
        S.fmt = FMT_CSR;
        S.lanes = L;
        std::vector<T> v(A.val.size());
        for (size_t k = 0; k < v.size(); ++k) v[k] = (T)A.val[k];
        S.rowptr = upload_vec(c, A.ptr);
        upload_csr_cols(c, S, A);
        S.val = upload_vec(c, v);
        consider(S, std::string("csr") + std::to_string(L) + (S.rbase ? "/r16" : S.d16 ? "/i16" : ""));
    }
    dev_free(c, x);
    dev_free(c, y);
    if (best.fmt == FMT_CSR)
        c->tune_record.push_back(key + "\tcsr " + std::to_string(best.lanes));
    else
        c->tune_record.push_back(key + "\tsell " + std::to_string(best.sell.lanes) + " " +
                                 std::to_string(best.sell.perm ? 1 : 0) + " " + std::to_string(best.sell.unroll));
    char line[200];
    const double fill = best.fmt == FMT_SELL && A.nnz() > 0 ? (double)best.sell.stored / (double)A.nnz() : 1.0;
    std::snprintf(line, sizeof line, "%s: %d x %d, %.1f nnz/row -> %s (%.1f us, stored/nnz %.2f)\n", what, A.n_rows,
                  A.n_cols, mean, best_name.c_str(), best_ms * 1e3, fill);
    c->tune_log += line;
    if (c->tune_verbose) c->tune_log += "  tried (us):" + tried + "\n";
    return best;
}

// A in CSR with L lanes per row.
template <typename T>
static SpMat<T> csr_spmat(eqs_ctx* c, const Csr<double>& A, int L) {
    SpMat<T> S;
    S.n_rows = A.n_rows; S.n_cols = A.n_cols; S.nnz = A.nnz();
    S.fmt = FMT_CSR;
    S.lanes = L;
    S.rowptr = upload_vec(c, A.ptr);
    upload_csr_cols(c, S, A);
    S.val = upload_vec(c, std::vector<T>(A.val.begin(), A.val.end()));
    return S;
}

// Values a_ij omega / a_jj of A omega D^{-1} in the storage order of the
// uploaded layout S of A (same structure, so the same positions).
template <typename T>
static T* scaled_values(eqs_ctx* c, const SpMat<T>& S, const Csr<double>& A, const std::vector<double>& d,
                        double omega) {
    Csr<double> As = A;
    for (size_t k = 0; k < As.val.size(); ++k) As.val[k] = A.val[k] * omega / d[A.col[k]];
    if (S.fmt == FMT_SELL) {  // the same layout (the row order depends on the pattern only)
        Sell<T> t = to_sell<T>(c, As, S.sell.lanes, S.sell.perm != nullptr);
        dev_free(c, t.sptr);
        dev_free(c, t.col);
        dev_free(c, t.d16);
        dev_free(c, t.pbase);
        dev_free(c, t.perm);
        return t.val;
    }
    std::vector<T> v(As.val.size());
    for (size_t k = 0; k < v.size(); ++k) v[k] = (T)As.val[k];
    return upload_vec(c, v);
}

// The finest level's Q: one lane per row (its kernel writes the CG partials of
// 256-row blocks). With `direct` it takes A_0's row order (or none), because
// one kernel walks both; else its own where that pays.
template <typename T>
static SpMat<T> finest_Q(eqs_ctx* c, const Csr<double>& Q, const Csr<double>& A0, bool direct, bool a0_sorted) {
    SpMat<T> S;
    S.n_rows = Q.n_rows; S.n_cols = Q.n_cols; S.nnz = Q.nnz();
    S.fmt = FMT_SELL;
    const bool sorted = direct ? a0_sorted : row_order_pays(Q);
    S.sell = to_sell<T>(c, Q, 1, sorted, direct ? &A0 : nullptr);
    S.sell.xcd = 1;  // with the finest smoothers' block order
    char line[160];
    std::snprintf(line, sizeof line, "Q0: %d x %d, %lld nonzeros, sell64%s (finest level), %s, stored/nnz %.2f\n", Q.n_rows,
                  Q.n_cols, (long long)Q.nnz(), sorted ? "s" : "", S.sell.d16 ? "16-bit column offsets" : "32-bit columns",
                  Q.nnz() ? (double)S.sell.stored / (double)Q.nnz() : 1.0);
    c->tune_log += line;
    return S;
}

// Q = P - w D^-1 (A P) = (I - w D^-1 A) P of a level (columns sorted per row):
// the prolongation with the post-smoother folded in, and, transposed, the
// restriction with the pre-smoother folded in, P^T (I - w A D^-1) (A symmetric).
static Csr<double> smoothed_prolongation(const Csr<double>& P, const Csr<double>& AP, const std::vector<double>& d,
                                         double w) {
    Csr<double> Q = AP;  // AP's pattern holds P's (A has its diagonal)
    for (int32_t i = 0; i < Q.n_rows; ++i) {
        int32_t e = P.ptr[i];
        for (int32_t k = Q.ptr[i]; k < Q.ptr[i + 1]; ++k) {
            double v = -w * AP.val[k] / d[i];
            if (e < P.ptr[i + 1] && P.col[e] == AP.col[k]) v += P.val[e++];
            Q.val[k] = v;
        }
        if (e != P.ptr[i + 1]) fail(EQS_ERR_INVALID_ARG, "AMG: prolongator entries outside A P");
    }
    return Q;
}

// Plain cycle: every level's A, P and R, the coarsest level's dense inverse.
template <typename T>
static void upload_plain(eqs_ctx* c, const AmgHost& ah, Hierarchy<T>& h) {
    const size_t L = ah.A.size();
    h.bottom = (int)L - 1;
    for (size_t l = 0; l < L; ++l) {
        Level<T>& lv = h.lv[l];
        // coarse operators may take a row order too: their smoothers write only rows of their own window
        lv.A = tuned_spmat<T>(c, ah.A[l], ("A" + std::to_string(l)).c_str(), l == 0, l > 0);
        std::vector<double> d = diagonal(ah.A[l]);
        std::vector<T> dinv(lv.n);
        for (int32_t i = 0; i < lv.n; ++i) dinv[i] = (T)(1.0 / d[i]);
        lv.dinv = upload_vec(c, dinv);
        for (T** q : {&lv.b, &lv.x, &lv.xs, &lv.res}) *q = (T*)dev_alloc(c, sizeof(T) * lv.n);
        if (l + 1 < L) {
            lv.sval = scaled_values<T>(c, lv.A, ah.A[l], d, lv.omega);
            lv.P = tuned_spmat<T>(c, ah.P[l], ("P" + std::to_string(l)).c_str(), false, true);
            lv.R = tuned_spmat<T>(c, ah.R[l], ("R" + std::to_string(l)).c_str(), false, true);
        } else {
            lv.dense_inv = upload_vec(c, std::vector<T>(ah.coarse_inv.begin(), ah.coarse_inv.end()));
        }
    }
}

// Up to this many finest rows the restriction is the folded Q_0^T on r itself:
// 8.8 entries per fine row (first-order stencil) against 7 + 3.6 in the
// pre-smoothing kernel and R_0, but one launch instead of two and one more
// product inside the last kernel. Small cycles are bound by the launches and
// their chains of dependent loads, large ones by the entries' bytes. RKC(8)
// steps, direct against pre-smoothed: 4.22 / 4.55 ms at 31,713 rows (FP32),
// 4.80 / 5.00 at 63,878 (FP64), 5.85 / 5.88 at 130,000 (FP32), 10.6 / 10.2
// (12 stages) at 266,175 (FP64).
constexpr int32_t kDirectRows = 100000;

// Folded cycle, formed here in FP64. A V(1,1) visit of a level l that is not
// the bottom is, with x = w D^-1 b, res = b - A x, x += P x_next,
// out = x + w D^-1 (b - A x):
//   b_next = P^T res = Q^T b,    out = G b + Q x_next,
//   Q = (I - w D^-1 A) P,        G = (2 I - w D^-1 A) w D^-1  (A's pattern),
// so two products replace pre-smoother, restriction, prolongation and
// post-smoother. Levels between the finest and the bottom hold Q^T and [G Q]
// (on the stacked vector [b; x_next]). The finest level's last kernel forms
// G r from the pre-smoothing values; large finest levels keep a pre-smoothing
// kernel, which writes w D^-1 (r + res) = G r and res, and restrict res.
// From the bottom level down the whole cycle is one dense symmetric matrix,
//   B_l = G_l + Q_l B_(l+1) Q_l^T  (the coarsest: its inverse),
// at the first level of at most 2 coarse_max (and kMaxBottom) unknowns; where
// that matrix times the restriction above it is small, the two are one.
template <typename T>
static void upload_folded(eqs_ctx* c, const AmgHost& ah, Hierarchy<T>& h) {
    const int L = (int)ah.A.size();
    int t = L - 1;
    for (int l = L - 1; l >= 1; --l)
        if (ah.A[l].n_rows <= std::min(kMaxBottom, 2 * c->amg.coarse_max)) t = l;
    h.folded = true;
    h.bottom = t;
    h.direct = ah.A[0].n_rows <= kDirectRows;
    std::vector<std::vector<double>> d(L);
    std::vector<Csr<double>> Q(L);
    for (int l = 0; l + 1 < L; ++l) {
        d[l] = diagonal(ah.A[l]);
        Q[l] = smoothed_prolongation(ah.P[l], ah.AP[l], d[l], ah.omega[l]);
    }
    auto g_value = [&](int l, int32_t i, int32_t e) {  // entry e (row i) of G_l
        const Csr<double>& A = ah.A[l];
        const int32_t j = A.col[e];
        const double w = ah.omega[l];
        return (j == i ? 2.0 * w / d[l][i] : 0.0) - w * w * A.val[e] / (d[l][i] * d[l][j]);
    };
    // the bottom's dense operator (symmetric)
    std::vector<double> B = ah.coarse_inv;
    for (int l = L - 2; l >= t; --l) {
        const int64_t n = ah.A[l].n_rows, m = ah.A[l + 1].n_rows;
        std::vector<double> W((size_t)(n * m), 0.0), Bl((size_t)(n * n), 0.0);  // W = Q B
        for (int64_t i = 0; i < n; ++i)
            for (int32_t e = Q[l].ptr[i]; e < Q[l].ptr[i + 1]; ++e)
                for (int64_t k = 0; k < m; ++k) W[(size_t)(i * m + k)] += Q[l].val[e] * B[(size_t)(Q[l].col[e] * m + k)];
        for (int64_t i = 0; i < n; ++i) {
            for (int64_t j = 0; j <= i; ++j) {
                double v = 0.0;
                for (int32_t e = Q[l].ptr[j]; e < Q[l].ptr[j + 1]; ++e) v += W[(size_t)(i * m + Q[l].col[e])] * Q[l].val[e];
                Bl[(size_t)(i * n + j)] = Bl[(size_t)(j * n + i)] = v;
            }
        }
        for (int32_t i = 0; i < (int32_t)n; ++i)
            for (int32_t e = ah.A[l].ptr[i]; e < ah.A[l].ptr[i + 1]; ++e) Bl[(size_t)i * n + ah.A[l].col[e]] += g_value(l, i, e);
        B.swap(Bl);
    }
    const int64_t nt = ah.A[t].n_rows, na = ah.A[t - 1].n_rows;
    h.small = h.direct && t == 1 && c->n_inst == 1 && small_solve_fits(c, na, ah.A[0].nnz(), nt, Q[0].nnz());
    const bool merged = !h.small && nt * na <= kMaxCoarseR;  // B_t times the restriction above it as one dense matrix
    Level<T>& bot = h.lv[t];
    if (merged) {
        const Csr<double>& up = (t > 1 || h.direct) ? Q[0 + (t - 1)] : ah.P[0];  // its transpose restricts
        std::vector<T> C((size_t)(nt * na));
        std::vector<double> row((size_t)na);
        for (int64_t i = 0; i < nt; ++i) {
            for (int64_t j = 0; j < na; ++j) {
                double v = 0.0;
                for (int32_t e = up.ptr[j]; e < up.ptr[j + 1]; ++e) v += B[(size_t)(i * nt + up.col[e])] * up.val[e];
                row[(size_t)j] = v;
            }
            for (int64_t j = 0; j < na; ++j) C[(size_t)(i * na + j)] = (T)row[(size_t)j];
        }
        bot.coarse_R = upload_vec(c, C);
        bot.coarse_R_cols = (int32_t)na;
    } else {
        bot.dense_inv = upload_vec(c, std::vector<T>(B.begin(), B.end()));
    }
    // vectors: b of every level below the finest, with the next level's result
    // behind it where a stacked product reads both
    for (int l = 1; l <= t; ++l) {
        const bool stacked = l < t;
        T* buf = (T*)dev_alloc(c, sizeof(T) * ((size_t)ah.A[l].n_rows + (stacked ? (size_t)ah.A[l + 1].n_rows : 0)));
        h.lv[l].b = buf;
        if (stacked) h.lv[l + 1].xs = buf + ah.A[l].n_rows;
    }
    h.lv[1].xs = (T*)dev_alloc(c, sizeof(T) * (size_t)ah.A[1].n_rows);
    for (int l = 0; l + 1 < L; ++l) {
        Level<T>& lv = h.lv[l];
        const std::string id = std::to_string(l);
        lv.A.nnz = ah.A[l].nnz();
        lv.P.nnz = ah.P[l].nnz();
        lv.R.nnz = ah.R[l].nnz();
        if (l >= t) continue;
        if (l == 0) {
            if constexpr (std::is_same_v<T, double>) lv.D = c->Mdia;  // A_0 is M
            else lv.D = to_dia<T>(c, ah.A[0]);
            std::vector<T> w(lv.n);
            for (int32_t i = 0; i < lv.n; ++i) w[i] = (T)(lv.omega / d[0][i]);
            lv.w = upload_vec(c, w);
            if (lv.D.K) {
                c->tune_log += "A0: " + std::to_string(lv.D.K) + " upper diagonals (finest level)\n";
            } else {
                Csr<double> As = ah.A[0];  // A w D^-1
                for (size_t k = 0; k < As.val.size(); ++k) As.val[k] *= lv.omega / d[0][As.col[k]];
                lv.A = tuned_spmat<T>(c, As, "A0", true);
                lv.sval = lv.A.sell.val;
            }
            if (!h.direct) {
                lv.x = (T*)dev_alloc(c, sizeof(T) * lv.n);
                lv.res = (T*)dev_alloc(c, sizeof(T) * lv.n);
            }
            // the direct form's last kernel walks A_0 and Q_0 with one row order
            lv.Q = finest_Q<T>(c, Q[0], ah.A[0], h.direct, lv.A.sell.perm != nullptr);
        } else {
            Csr<double> GQ;
            const int32_t n = ah.A[l].n_rows;
            GQ.n_rows = n;
            GQ.n_cols = n + ah.A[l + 1].n_rows;
            GQ.ptr.assign((size_t)n + 1, 0);
            GQ.col.reserve((size_t)(ah.A[l].nnz() + Q[l].nnz()));
            GQ.val.reserve((size_t)(ah.A[l].nnz() + Q[l].nnz()));
            for (int32_t i = 0; i < n; ++i) {
                for (int32_t e = ah.A[l].ptr[i]; e < ah.A[l].ptr[i + 1]; ++e) {
                    GQ.col.push_back(ah.A[l].col[e]);
                    GQ.val.push_back(g_value(l, i, e));
                }
                for (int32_t e = Q[l].ptr[i]; e < Q[l].ptr[i + 1]; ++e) {
                    GQ.col.push_back(n + Q[l].col[e]);
                    GQ.val.push_back(Q[l].val[e]);
                }
                GQ.ptr[(size_t)i + 1] = (int32_t)GQ.col.size();
            }
            lv.GQ = tuned_spmat<T>(c, GQ, ("[G Q]" + id).c_str(), false, true, GQ.n_rows);
        }
        if (l == t - 1 && merged) continue;
        if (h.small) {
            lv.R = csr_spmat<T>(c, transpose(Q[l]), 16);
            c->tune_log += "R0(I-AwD^-1): csr16 (small system: solves in one launch)\n";
        } else if (l > 0 || h.direct)
            lv.R = tuned_spmat<T>(c, transpose(Q[l]), ("R" + id + "(I-AwD^-1)").c_str(), false, true);
        else
            lv.R = tuned_spmat<T>(c, ah.R[l], ("R" + id).c_str(), false, true);
    }
}

template <typename T>
static void upload_hierarchy(eqs_ctx* c, const AmgHost& ah, Hierarchy<T>& h) {
    h = Hierarchy<T>{};
    h.lv.resize(ah.A.size());
    for (size_t l = 0; l < ah.A.size(); ++l) {
        h.lv[l].n = ah.A[l].n_rows;
        h.lv[l].A.nnz = ah.A[l].nnz();
        h.lv[l].omega = ah.omega[l];
    }
    if (c->fold && ah.A.size() > 1) upload_folded<T>(c, ah, h);
    else upload_plain<T>(c, ah, h);
}

// Morton key of a point quantised to 21 bits per axis inside the box [lo, hi].
static uint64_t morton3(const double* p, const double* lo, const double* inv_ext) {
    uint64_t key = 0;
    uint32_t q[3];
    for (int d = 0; d < 3; ++d) {
        double f = (p[d] - lo[d]) * inv_ext[d];
        f = std::min(std::max(f, 0.0), 1.0);
        q[d] = (uint32_t)(f * 2097151.0);
    }
    for (int bit = 20; bit >= 0; --bit)
        for (int d = 0; d < 3; ++d) key = (key << 1) | ((q[d] >> bit) & 1u);
    return key;
}

// Element blocks for the fused element pass: tets sorted by instance, then by
// the Morton code of their centroid, cut into blocks of kTetBlock * tpt tets;
// per block the sorted distinct internal node ids and, per tet, a 64-bit
// record: 16-bit material, then the four 12-bit block-local vertex ids.
struct ElementBlocks {
    std::vector<uint64_t> pack;
    std::vector<int32_t> boff, bnodes;
    int32_t max_nodes = 0;
};

static std::vector<int32_t> morton_tet_order(const eqs_ctx* c) {
    const int64_t T = c->n_tets;
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
    for (int64_t i = 0; i < c->n_nodes; ++i)
        for (int d = 0; d < 3; ++d) {
            lo[d] = std::min(lo[d], c->xyz[3 * i + d]);
            hi[d] = std::max(hi[d], c->xyz[3 * i + d]);
        }
    double inv_ext[3];
    for (int d = 0; d < 3; ++d) inv_ext[d] = hi[d] > lo[d] ? 1.0 / (hi[d] - lo[d]) : 0.0;
    std::vector<std::pair<uint64_t, int32_t>> key(T);
    std::vector<int32_t> tinst(T, 0);
    for (int64_t i = 0; i < c->n_inst; ++i)
        for (int64_t e = c->inst_tet_off[i]; e < c->inst_tet_off[i + 1]; ++e) tinst[e] = (int32_t)i;
    for (int64_t e = 0; e < T; ++e) {
        double cen[3] = {0, 0, 0};
        for (int a = 0; a < 4; ++a)
            for (int d = 0; d < 3; ++d) cen[d] += 0.25 * c->xyz[3 * (int64_t)c->tets[(int64_t)c->npe * e + a] + d];
        key[e] = {morton3(cen, lo, inv_ext), (int32_t)e};
    }
    // instance first (blocks then never mix instances, whose meshes may overlap in space)
    std::stable_sort(key.begin(), key.end(),
                     [&](const std::pair<uint64_t, int32_t>& x, const std::pair<uint64_t, int32_t>& y) {
                         if (tinst[x.second] != tinst[y.second]) return tinst[x.second] < tinst[y.second];
                         return x.first < y.first;
                     });
    std::vector<int32_t> order(T);
    for (int64_t k = 0; k < T; ++k) order[k] = key[k].second;
    return order;
}

// Second-order tets take two 64-bit words per record: 16-bit material, then
// the ten 11-bit block-local ids at bits 16 + 11 k of the 128-bit pair (low
// word first).
static ElementBlocks element_blocks(const eqs_ctx* c, const std::vector<int32_t>& u2i,
                                    const std::vector<int32_t>& order, int tpt) {
    const int64_t T = c->n_tets, per = (int64_t)kTetBlock * tpt;
    const int64_t nb = (T + per - 1) / per;
    const int npe = c->npe, words = npe == 4 ? 1 : 2;
    ElementBlocks eb;
    eb.pack.assign((size_t)(nb * per * words), ~0ull);  // whole blocks; padding records are skipped
    eb.boff.assign(nb + 1, 0);
    eb.bnodes.reserve((size_t)T);
    std::vector<int32_t> ids;
    for (int64_t b = 0; b < nb; ++b) {
        const int64_t e0 = b * per, e1 = std::min<int64_t>(T, e0 + per);
        ids.clear();
        for (int64_t k = e0; k < e1; ++k)
            for (int a = 0; a < npe; ++a) ids.push_back(u2i[c->tets[npe * (int64_t)order[k] + a]]);
        std::sort(ids.begin(), ids.end());
        ids.erase(std::unique(ids.begin(), ids.end()), ids.end());
        if (ids.size() > (size_t)kMaxBlockNodes) {  // local ids / LDS: the caller tries a smaller block
            eb.max_nodes = INT32_MAX;
            return eb;
        }
        eb.max_nodes = std::max<int32_t>(eb.max_nodes, (int32_t)ids.size());
        for (int64_t k = e0; k < e1; ++k) {
            const int32_t e = order[k];
            uint64_t w = (uint64_t)(uint16_t)c->tet_mat[e], w2 = 0;
            for (int a = 0; a < npe; ++a) {
                const uint64_t loc =
                    (uint64_t)(std::lower_bound(ids.begin(), ids.end(), u2i[c->tets[npe * (int64_t)e + a]]) - ids.begin());
                if (npe == 4) {
                    w |= loc << (16 + 12 * a);
                } else {
                    const int pos = 16 + 11 * a;
                    if (pos < 64) w |= loc << pos;
                    if (pos + 11 > 64) w2 |= pos >= 64 ? loc << (pos - 64) : loc >> (64 - pos);
                }
            }
            eb.pack[k * words] = w;
            if (words == 2) eb.pack[k * words + 1] = w2;
        }
        eb.bnodes.insert(eb.bnodes.end(), ids.begin(), ids.end());
        if (eb.bnodes.size() > (size_t)INT32_MAX) fail(EQS_ERR_INVALID_ARG, "too many block nodes");
        eb.boff[b + 1] = (int32_t)eb.bnodes.size();
    }
    return eb;
}

// Fans of the element pass (k_kx_fan): tets of one material around a common edge,
// each sharing a face with the next. Tets are grouped by their longest edge (the
// body diagonal of every cube of a Kuhn mesh, whose six tets are one ring) within
// windows of the Morton order, a group is walked into chains, and chains are cut
// into fans of at most kFanTets; half as long where tets are taken one by one
// (single[material]), so that no thread has six exp(alpha ln r) in a row. Order of
// the fans: their first tet's.
struct Fan {
    int32_t first;  // position of its first tet in the Morton order
    int32_t mat, count;
    int32_t node[9];  // a, b, r_0 .. r_count (internal ids)
};
static std::vector<Fan> build_fans(const eqs_ctx* c, const std::vector<int32_t>& u2i, const std::vector<int32_t>& order,
                                   const std::vector<char>& single) {
    constexpr int64_t kWindow = 1 << 18;
    static const int ev[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
    static const int opp[6][2] = {{2, 3}, {1, 3}, {1, 2}, {0, 3}, {0, 2}, {0, 1}};
    const int64_t T = c->n_tets;
    std::vector<Fan> fans;
    fans.reserve((size_t)(T / 4));
    struct Item {
        uint64_t edge;
        int32_t mat, pos, r, s;
    };
    std::vector<Item> it;
    std::vector<char> used;
    for (int64_t w0 = 0; w0 < T; w0 += kWindow) {
        const int64_t w1 = std::min<int64_t>(T, w0 + kWindow);
        it.clear();
        for (int64_t k = w0; k < w1; ++k) {
            const int32_t e = order[k];
            const int32_t* v = &c->tets[4 * (int64_t)e];
            int32_t id[4];
            for (int a = 0; a < 4; ++a) id[a] = u2i[v[a]];
            int best = 0;
            double bl = -1.0;
            uint64_t bkey = 0;
            for (int q = 0; q < 6; ++q) {
                const double* p0 = &c->xyz[3 * (int64_t)v[ev[q][0]]];
                const double* p1 = &c->xyz[3 * (int64_t)v[ev[q][1]]];
                double l = 0.0;
                for (int d = 0; d < 3; ++d) l += (p1[d] - p0[d]) * (p1[d] - p0[d]);
                const uint32_t i0 = (uint32_t)id[ev[q][0]], i1 = (uint32_t)id[ev[q][1]];
                const uint64_t key = ((uint64_t)std::min(i0, i1) << 32) | std::max(i0, i1);
                // equal lengths (up to rounding): the smaller key, the same for every tet of the edge
                if (l > bl * (1.0 + 1e-9) || (l >= bl * (1.0 - 1e-9) && key < bkey)) {
                    best = q;
                    bl = std::max(l, bl);
                    bkey = key;
                }
            }
            it.push_back(Item{bkey, c->tet_mat[e], (int32_t)k, id[opp[best][0]], id[opp[best][1]]});
        }
        std::sort(it.begin(), it.end(), [](const Item& x, const Item& y) {
            if (x.edge != y.edge) return x.edge < y.edge;
            if (x.mat != y.mat) return x.mat < y.mat;
            return x.pos < y.pos;
        });
        for (size_t g0 = 0, g1; g0 < it.size(); g0 = g1) {
            for (g1 = g0; g1 < it.size() && it[g1].edge == it[g0].edge && it[g1].mat == it[g0].mat;) ++g1;
            used.assign(g1 - g0, 0);
            auto other_use = [&](int32_t r, size_t me) {  // another unused tet of the group with node r
                for (size_t k = g0; k < g1; ++k)
                    if (k != me && !used[k - g0] && (it[k].r == r || it[k].s == r)) return (int64_t)k;
                return (int64_t)-1;
            };
            for (size_t left = g1 - g0; left > 0;) {
                // a chain's end: an unused tet with a face that no other one shares; else (a ring) any
                size_t st = g1;
                int32_t from = -1;
                for (size_t k = g0; k < g1 && from < 0; ++k) {
                    if (used[k - g0]) continue;
                    if (st == g1) st = k;
                    if (other_use(it[k].r, k) < 0) { st = k; from = it[k].r; }
                    else if (other_use(it[k].s, k) < 0) { st = k; from = it[k].s; }
                }
                if (from < 0) from = it[st].r;
                Fan f{};
                f.mat = it[st].mat;
                f.node[0] = (int32_t)(it[st].edge >> 32);
                f.node[1] = (int32_t)(it[st].edge & 0xffffffffu);
                f.node[2] = from;
                f.first = it[st].pos;
                int64_t k = (int64_t)st;
                while (k >= 0 && f.count < (single[f.mat] ? kFanTets / 2 : kFanTets)) {
                    used[(size_t)k - g0] = 1;
                    --left;
                    from = it[(size_t)k].r == from ? it[(size_t)k].s : it[(size_t)k].r;
                    f.node[3 + f.count++] = from;
                    f.first = std::min(f.first, it[(size_t)k].pos);
                    k = other_use(from, (size_t)k);
                }
                fans.push_back(f);
            }
        }
    }
    std::stable_sort(fans.begin(), fans.end(), [](const Fan& x, const Fan& y) { return x.first < y.first; });
    return fans;
}

// Blocks of kTetBlock fans, those taken tet by tet (single[material]) last, so that
// few wavefronts have both kinds: words material | a | b | r_0 | r_1 and
// r_2 .. r_6 | count (12-bit block-local ids; ids past the fan repeat its last).
static ElementBlocks fan_blocks(std::vector<Fan>& fans, const std::vector<char>& single) {
    const int64_t F = (int64_t)fans.size(), nb = (F + kTetBlock - 1) / kTetBlock;
    ElementBlocks eb;
    eb.pack.assign((size_t)(nb * kTetBlock * 2), 0);
    eb.boff.assign(nb + 1, 0);
    eb.bnodes.reserve((size_t)F);
    std::vector<int32_t> ids;
    for (int64_t b = 0; b < nb; ++b) {
        const int64_t f0 = b * kTetBlock, f1 = std::min<int64_t>(F, f0 + kTetBlock);
        ids.clear();
        std::stable_partition(fans.begin() + f0, fans.begin() + f1, [&](const Fan& f) { return !single[f.mat]; });
        for (int64_t f = f0; f < f1; ++f) ids.insert(ids.end(), fans[f].node, fans[f].node + 3 + fans[f].count);
        std::sort(ids.begin(), ids.end());
        ids.erase(std::unique(ids.begin(), ids.end()), ids.end());
        if (ids.size() > (size_t)kMaxBlockNodes) {
            eb.max_nodes = INT32_MAX;
            return eb;
        }
        eb.max_nodes = std::max<int32_t>(eb.max_nodes, (int32_t)ids.size());
        for (int64_t f = f0; f < f1; ++f) {
            const Fan& a = fans[f];
            uint64_t loc[9];
            for (int k = 0; k < 9; ++k) {
                const int32_t id = a.node[std::min(k, 2 + a.count)];
                loc[k] = (uint64_t)(std::lower_bound(ids.begin(), ids.end(), id) - ids.begin());
            }
            eb.pack[2 * f] = (uint64_t)(uint16_t)a.mat | loc[0] << 16 | loc[1] << 28 | loc[2] << 40 | loc[3] << 52;
            eb.pack[2 * f + 1] = loc[4] | loc[5] << 12 | loc[6] << 24 | loc[7] << 36 | loc[8] << 48 | (uint64_t)a.count << 60;
        }
        eb.bnodes.insert(eb.bnodes.end(), ids.begin(), ids.end());
        if (eb.bnodes.size() > (size_t)INT32_MAX) fail(EQS_ERR_INVALID_ARG, "too many block nodes");
        eb.boff[b + 1] = (int32_t)eb.bnodes.size();
    }
    return eb;
}

// Lists of the deterministic element pass (k_kx_det, k_kx_gather) from the
// blocks: slot 4 t + a is vertex a of the block's record t; a node's slots and
// a node's block occurrences are listed in increasing order (counting sorts).
static void install_det_lists(eqs_ctx* c, const ElementBlocks& eb, int tpt) {
    const int64_t nb = c->n_blocks, per = (int64_t)kTetBlock * tpt, NB = (int64_t)eb.bnodes.size();
    std::vector<uint16_t> kslots((size_t)(nb * per * 4), 0), kend((size_t)NB, 0);
    std::vector<int32_t> pos;
    for (int64_t b = 0; b < nb; ++b) {
        const int32_t off = eb.boff[b], nn = eb.boff[b + 1] - off;
        pos.assign((size_t)nn + 1, 0);
        for (int64_t t = 0; t < per; ++t) {
            const uint64_t w = eb.pack[(size_t)(b * per + t)];
            if (w == ~0ull) continue;
            for (int a = 0; a < 4; ++a) pos[((w >> (16 + 12 * a)) & 0xfffu) + 1]++;
        }
        for (int32_t k = 0; k < nn; ++k) {
            pos[k + 1] += pos[k];
            kend[(size_t)(off + k)] = (uint16_t)pos[k + 1];
        }
        uint16_t* sl = kslots.data() + b * per * 4;
        for (int64_t t = 0; t < per; ++t) {
            const uint64_t w = eb.pack[(size_t)(b * per + t)];
            if (w == ~0ull) continue;
            for (int a = 0; a < 4; ++a) sl[pos[(w >> (16 + 12 * a)) & 0xfffu]++] = (uint16_t)(4 * t + a);
        }
    }
    std::vector<int32_t> occ_off((size_t)c->n_nodes + 1, 0), occ((size_t)NB);
    for (int64_t p = 0; p < NB; ++p) occ_off[(size_t)eb.bnodes[p] + 1]++;
    for (int64_t i = 0; i < c->n_nodes; ++i) occ_off[i + 1] += occ_off[i];
    std::vector<int32_t> fill(occ_off.begin(), occ_off.end() - 1);
    for (int64_t p = 0; p < NB; ++p) occ[(size_t)fill[eb.bnodes[p]]++] = (int32_t)p;
    c->d_kslots = upload_vec(c, kslots);
    c->d_kend = upload_vec(c, kend);
    c->d_occ_off = upload_vec(c, occ_off);
    c->d_occ = upload_vec(c, occ);
    c->d_kx_part = (double*)dev_alloc(c, sizeof(double) * (size_t)std::max<int64_t>(NB, 1));
}

// tpt 0: eb holds fans
static void install_blocks(eqs_ctx* c, const ElementBlocks& eb, int tpt) {
    if (c->d_tpack) { dev_free(c, c->d_tpack); dev_free(c, c->d_bnodes); dev_free(c, c->d_boff); }
    if (c->d_kslots) {
        for (void* q : {(void*)c->d_kslots, (void*)c->d_kend, (void*)c->d_occ_off, (void*)c->d_occ, (void*)c->d_kx_part})
            dev_free(c, q);
        c->d_kslots = nullptr; c->d_kend = nullptr; c->d_occ_off = nullptr; c->d_occ = nullptr; c->d_kx_part = nullptr;
    }
    c->n_blocks = (int64_t)eb.boff.size() - 1;
    c->max_block_nodes = eb.max_nodes;
    c->n_block_nodes = (int64_t)eb.bnodes.size();
    c->tet_tpt = tpt;
    c->fans = tpt == 0;
    c->d_tpack = upload_vec(c, eb.pack);
    c->d_bnodes = upload_vec(c, eb.bnodes);
    c->d_boff = upload_vec(c, eb.boff);
    if (c->deterministic) {
        if (c->npe != 4) fail(EQS_ERR_INVALID_ARG, "the deterministic element pass is built for first-order tets");
        install_det_lists(c, eb, tpt);
    }
}

static int32_t int_exponent(double alpha) {
    return (alpha == std::floor(alpha) && alpha >= 0 && alpha <= 64) ? (int32_t)alpha : -1;
}

// Fans where they hold most of a ring and their blocks fill the chip (some 3 per
// CU): stage_rhs with its fill takes 28.0 us against 26.9 with the best
// block of single tets at 750,000 tets, 31.1 | 31.0 at 1.3M, 31.9 | 32.1 at 1.6M,
// 38.8 | 41.7 at 2.6M, 89.3 | 93.2 at 12.6M. No block size is timed then, which
// takes half of the build's time off (12.6M tets: 7.7 instead of 12.7 s).
constexpr double kMinFanLength = 4.0;
constexpr int64_t kMinFans = 800 * kTetBlock;
// The deterministic pass has lists for single tets. Tets whose exponent is no
// whole number are taken one by one also inside a fan, so a mesh with many of them
// stays with single tets.
static bool fans_apply(const eqs_ctx* c, const std::vector<char>& single) {
    if (c->npe != 4 || c->deterministic || !c->fan_pass || c->n_tets < 2 * kMinFans) return false;
    int64_t n = 0;
    for (int64_t e = 0; e < c->n_tets; ++e) n += single[c->tet_mat[e]];
    return 4 * n <= c->n_tets;
}

// Blocks of 256 tets per workgroup trade LDS reuse (each block re-reads the
// nodes it shares with its neighbours) against parallelism; with autotuning
// on, every block size that fits the local ids is timed on the RHS pass and
// the fastest kept (else 4 tets per thread). Large first-order meshes take fans.
void build_element_blocks(eqs_ctx* c, const std::vector<int32_t>& u2i, const double* yfree, double* out) {
    const std::vector<int32_t> order = morton_tet_order(c);
    const int fixed = c->npe == 4 ? 4 : 1;
    const std::string key = "element " + std::to_string(c->n_tets) + " " + std::to_string(c->npe);
    const auto rec = c->autotune ? c->tune_replay.find(key) : c->tune_replay.end();
    const bool replay = rec != c->tune_replay.end();
    std::vector<char> single(c->mats.size(), 0);
    for (size_t m = 0; m < c->mats.size(); ++m) single[m] = c->mats[m].nonlinear && int_exponent(c->mats[m].alpha) < 0;
    if (fans_apply(c, single) && (!replay || rec->second == "fans")) {
        std::vector<Fan> fans = build_fans(c, u2i, order, single);
        const double len = (double)c->n_tets / (double)fans.size();
        const ElementBlocks eb = len >= kMinFanLength && (int64_t)fans.size() >= kMinFans ? fan_blocks(fans, single) : ElementBlocks{};
        if (!eb.boff.empty() && eb.max_nodes <= kMaxBlockNodes) {
            install_blocks(c, eb, 0);
            char buf[96];
            std::snprintf(buf, sizeof buf, "element: %d fans per block (%.2f tets a fan)%s\n", kTetBlock, len,
                          replay ? " (tuning record)" : "");
            c->tune_log += buf;
            if (c->autotune) c->tune_record.push_back(key + "\tfans");
            return;
        }
    }
    // a record of fans where this context takes none: the block size that needs no timing, the same every time
    const bool untimed = replay && rec->second == "fans";
    if (!c->autotune || untimed || c->n_tets < 16 * (int64_t)kTetBlock * kMaxTetsPerThread) {
        for (int tpt = fixed; tpt >= 1; tpt /= 2) {
            ElementBlocks eb = element_blocks(c, u2i, order, tpt);
            if (eb.max_nodes <= kMaxBlockNodes) {
                install_blocks(c, eb, tpt);
                c->tune_log += "element: " + std::to_string(kTetBlock * tpt) + " tets per block" +
                               (untimed ? " (tuning record)\n" : "\n");
                return;
            }
        }
        fail(EQS_ERR_INVALID_ARG, "element block of 256 tets with more than " + std::to_string(kMaxBlockNodes) +
                                      " distinct nodes");
    }
    {
        if (replay) {  // a recorded block size
            const int tpt = std::atoi(rec->second.c_str());
            if (tpt < 1 || tpt > kMaxTetsPerThread || (tpt & (tpt - 1)))
                fail(EQS_ERR_INVALID_ARG, "tuning record: bad entry for " + key + ": " + rec->second);
            ElementBlocks eb = element_blocks(c, u2i, order, tpt);
            if (eb.max_nodes > kMaxBlockNodes) fail(EQS_ERR_INVALID_ARG, "tuning record: " + key + " does not fit");
            install_blocks(c, eb, tpt);
            c->tune_log += "element: " + std::to_string(kTetBlock * tpt) + " tets per block (tuning record)\n";
            return;
        }
    }
    int best_tpt = 0;
    double best = 1e300;
    std::string line = "element:";
    const int max_tpt = c->npe == 4 ? kMaxTetsPerThread : 2;  // second order: ~1.3 nodes per tet
    for (int tpt = 1; tpt <= max_tpt; tpt *= 2) {
        ElementBlocks eb = element_blocks(c, u2i, order, tpt);
        if (eb.max_nodes > kMaxBlockNodes) break;
        install_blocks(c, eb, tpt);
        const double ms = time_kx(c, yfree, out, 5);
        char buf[64];
        std::snprintf(buf, sizeof buf, " %d:%.1fus", kTetBlock * tpt, 1e3 * ms);
        line += buf;
        if (ms < best) {
            best = ms;
            best_tpt = tpt;
        }
    }
    if (best_tpt == 0)
        fail(EQS_ERR_INVALID_ARG, "element block of 256 tets with more than " + std::to_string(kMaxBlockNodes) +
                                      " distinct nodes");
    if (best_tpt != c->tet_tpt) install_blocks(c, element_blocks(c, u2i, order, best_tpt), best_tpt);
    c->tune_log += line + " -> " + std::to_string(kTetBlock * best_tpt) + " tets per block\n";
    c->tune_record.push_back(key + "\t" + std::to_string(best_tpt));
}

void upload(eqs_ctx* c) {
    const int64_t N = c->n_nodes, T = c->n_tets, NF = c->n_free;
    std::vector<int32_t> u2i(N);
    for (int64_t i = 0; i < N; ++i) u2i[c->int_to_user[i]] = (int32_t)i;

    std::vector<double> px(N), py(N), pz(N);
    for (int64_t i = 0; i < N; ++i) {
        const double* p = &c->xyz[3 * (int64_t)c->int_to_user[i]];
        px[i] = p[0];
        py[i] = p[1];
        pz[i] = p[2];
    }
    std::vector<MatDev> md(c->mats.size());
    for (size_t m = 0; m < c->mats.size(); ++m) {
        const eqs_material& s = c->mats[m];
        md[m].eps = kEps0 * s.eps_r;
        md[m].kappa0 = s.kappa0;
        md[m].inv_es = s.nonlinear ? 1.0 / s.e_s : 0.0;
        md[m].alpha = s.alpha;
        md[m].nonlinear = s.nonlinear ? 1 : 0;
        md[m].ialpha = int_exponent(s.alpha);
    }
    std::vector<int32_t> dd(c->n_dir);
    {
        std::vector<int32_t> drive_of(N, -1);
        for (size_t k = 0; k < c->dir_nodes.size(); ++k) drive_of[c->dir_nodes[k]] = c->dir_drive[k];
        for (int64_t k = 0; k < c->n_dir; ++k) dd[k] = drive_of[c->int_to_user[NF + k]];
    }
    c->d_cx = upload_vec(c, px);
    c->d_cy = upload_vec(c, py);
    c->d_cz = upload_vec(c, pz);
    c->d_mats = upload_vec(c, md);
    c->d_ddrive = upload_vec(c, dd);
    {
        std::vector<DriveDev> dr(c->drives.size());
        for (size_t k = 0; k < dr.size(); ++k)
            dr[k] = DriveDev{2.0 * M_PI * c->drives[k].freq, c->drives[k].amp, c->drives[k].phase, 0.0};
        c->d_drives = upload_vec(c, dr);
    }
    c->d_int_to_user = upload_vec(c, c->int_to_user);

    c->tune_log.clear();
    Csr<double> M = assemble_M_free(c);
    c->nnz_M = M.nnz();
    c->M = to_sell<double>(c, M, 1, row_order_pays(M));
    c->M.xcd = 1;  // the CG SpMV walks its row blocks in the XCD order (row_block in sell.h)
    c->Mdia = to_dia<double>(c, M);
    c->tune_log += std::string("M: sell64") + (c->M.perm ? "s (rows sorted within 256-row windows)" : "") + ", " +
                   (c->M.d16 ? "16-bit column offsets" : "32-bit columns") +
                   (c->Mdia.K ? "; in CG " + std::to_string(c->Mdia.K) + " upper diagonals\n" : "\n");
    AmgHost ah = build_sa_amg(M, c->amg, c->fold);
    if (c->amg.precision == EQS_PREC_FP32) upload_hierarchy<float>(c, ah, c->h32);
    else upload_hierarchy<double>(c, ah, c->h64);

    auto vec = [&](int64_t n) { return (double*)dev_alloc(c, sizeof(double) * (size_t)n); };
    c->d_r = vec(NF); c->d_z = vec(NF); c->d_p = vec(NF); c->d_q = vec(NF); c->d_mx = vec(NF);
    c->mx_of_F = false;
    c->d_Y0 = vec(NF); c->d_Ya = vec(NF); c->d_Yb = vec(NF); c->d_Yc = vec(NF); c->d_F0 = vec(NF); c->d_F = vec(NF);
    c->d_rhs = vec(NF); c->d_rhs_alt = vec(NF); c->d_tmpN = vec(N); c->d_tmpN2 = vec(N);
    c->max_blocks = (std::max<int64_t>(N, T) + kBlock - 1) / kBlock + 1;
    c->d_partials = vec(12 * c->max_blocks);
    c->d_scal = (PcgScalars*)dev_alloc(c, sizeof(PcgScalars) * (size_t)c->n_inst);
    c->d_step = (PcgStep*)dev_alloc(c, sizeof(PcgStep) * (size_t)c->n_inst);
    EQS_HIP(hipMemset(c->d_step, 0, sizeof(PcgStep) * (size_t)c->n_inst));
    c->d_sum = (PcgSummary*)dev_alloc(c, sizeof(PcgSummary));
    EQS_HIP(hipMemset(c->d_sum, 0, sizeof(PcgSummary)));
    c->d_force = (int32_t*)dev_alloc(c, sizeof(int32_t));
    EQS_HIP(hipMemset(c->d_force, 0, sizeof(int32_t)));
    EQS_HIP(hipHostMalloc((void**)&c->h_scal, sizeof(PcgScalars) * (size_t)c->n_inst, hipHostMallocMapped));
    EQS_HIP(hipHostGetDevicePointer((void**)&c->d_hscal, c->h_scal, 0));
    EQS_HIP(hipHostMalloc((void**)&c->h_sum, sizeof(PcgSummary), hipHostMallocMapped));
    EQS_HIP(hipHostGetDevicePointer((void**)&c->d_hsum, c->h_sum, 0));
    c->d_inst_row = upload_vec(c, c->inst_row_off);
    {
        const int64_t nb = (NF + kBlock - 1) / kBlock;
        std::vector<int32_t> bi(std::max<int64_t>(nb, 1), 0);
        int32_t i = 0;
        for (int64_t b = 0; b < nb; ++b) {
            while (i + 1 < c->n_inst && c->inst_row_off[i + 1] <= b * kBlock) ++i;
            bi[b] = i;
        }
        c->d_blk_inst = upload_vec(c, bi);
    }
    guess_alloc_scratch(c);  // eqs_galerkin_start's dot scratch
    launch_fill(c->stream, c->d_Y0, 0.0, NF);
    build_element_blocks(c, u2i, c->d_Y0, c->d_rhs);
    if (!c->tune_file.empty() && c->tune_replay.empty() && c->autotune) {
        FILE* f = std::fopen(c->tune_file.c_str(), "w");
        if (!f) fail(EQS_ERR_INVALID_ARG, "tuning record: cannot write " + c->tune_file);
        // a line without a tab is no entry: a build that timed nothing leaves a record all the
        // same, and the next one that does replaces it
        if (c->tune_record.empty()) std::fprintf(f, "# every layout of this build follows from sizes\n");
        for (const std::string& ln : c->tune_record) std::fprintf(f, "%s\n", ln.c_str());
        std::fclose(f);
    }
    c->tune_record.clear();
    EQS_HIP(hipEventCreateWithFlags(&c->ev[0], hipEventDisableTiming));
    EQS_HIP(hipEventCreateWithFlags(&c->ev[1], hipEventDisableTiming));
    c->have_Flast = false;
}

void free_device(eqs_ctx* c) {
    if (c->guess.tstream) (void)hipStreamSynchronize(c->guess.tstream);
    release_graphs(c);
    // the network's buffers belong to this memory too
    if (c->guess.net) {
        mlp_destroy(c->guess.net);
        c->guess.net = nullptr;
    }
    for (auto& a : c->allocations)
        if (!in_workspace(c, a.first)) (void)hipFree(a.first);
    c->allocations.clear();
    c->device_bytes = 0;
    ws_reset(c);  // a workspace stays attached, empty
    if (c->h_scal) { (void)hipHostFree(c->h_scal); c->h_scal = nullptr; c->d_hscal = nullptr; }
    if (c->h_dots) { (void)hipHostFree(c->h_dots); c->h_dots = nullptr; c->d_hdots = nullptr; }
    if (c->h_sum) { (void)hipHostFree(c->h_sum); c->h_sum = nullptr; c->d_hsum = nullptr; }
    c->d_sum = nullptr; c->d_inst_row = nullptr; c->d_blk_inst = nullptr; c->d_force = nullptr;
    for (auto& e : c->ev)
        if (e) { (void)hipEventDestroy(e); e = nullptr; }
    c->M = Sell<double>{};
    c->Mdia = Dia<double>{};
    c->stage_iters.clear();
    c->h64 = Hierarchy<double>{};
    c->h32 = Hierarchy<float>{};
    c->d_tpack = nullptr; c->d_bnodes = nullptr; c->d_boff = nullptr; c->n_blocks = 0; c->max_block_nodes = 0; c->n_block_nodes = 0;
    c->d_kslots = nullptr; c->d_kend = nullptr; c->d_occ_off = nullptr; c->d_occ = nullptr; c->d_kx_part = nullptr;
    c->d_cx = c->d_cy = c->d_cz = nullptr; c->d_mats = nullptr; c->tet_tpt = 0; c->fans = false;
    c->d_ddrive = nullptr; c->d_int_to_user = nullptr; c->d_drives = nullptr;
    c->d_r = c->d_z = c->d_p = c->d_q = c->d_mx = nullptr;
    c->mx_of_F = false;
    c->d_Y0 = c->d_Ya = c->d_Yb = c->d_Yc = c->d_F0 = c->d_F = nullptr;
    c->d_rhs = c->d_rhs_alt = c->d_tmpN = c->d_tmpN2 = nullptr;
    c->d_partials = nullptr;
    c->d_scal = nullptr;
    c->d_step = nullptr;
    c->built = false;
    c->have_Flast = false;
    c->guess.dev_ready = false;
    c->guess.d_S = c->guess.d_rprev = c->guess.d_alpha = c->guess.d_part = nullptr;
    c->guess.d_guard = nullptr;
    c->guess.d_gstat = nullptr;
    c->guess.d_bx = c->guess.d_bt = nullptr;
    if (!c->guess.G.empty()) guess_reset(c);
}

}  // namespace eqs
