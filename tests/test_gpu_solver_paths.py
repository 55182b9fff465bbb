"""The CG solve's forms against each other and against the FP64 oracle's M:

* small single systems in one launch (EQS_SMALL=0: by launches),
* the finest matrices by diagonals (EQS_DIAGONALS=0: sliced rows), with 3
  diagonals (Kuhn mesh) and 7 (its nodes moved), alone and in a batch,
* the reductions taken by the next kernel or by finaliser launches (timing the
  finaliser class asks for those), on few and on many row blocks,
* the restriction of the finest level taken with the residual, on either side
  of the row count where it ends.

Environment switches are read when a context is created. Each form solves to
the same true residual: |b - M x| <= rtol |b|, checked here with the oracle's
matrix; the bound gets 1e-14 for that product's own rounding (15 terms of
relative 2^-53 each, of a size |M||x| within 1e1 of |b| here). Forms differ in
rounding only, so the iteration counts agree up to one.
"""

import numpy as np
import pytest

import eqsgen
from oracle.eqs import EqsOracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1612_09447_amd import EQS_PREC_FP32, EQS_PREC_FP64, Batch, Context, EqsError  # noqa: E402

DEV = torch.device("cuda:0")
RTOL = 1e-11


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


def moved(case, seed=2):
    """Inner nodes moved by up to a tenth of a cell: M gets all of the mesh's edges."""
    h = 0.1 / case.n
    inner = np.all((case.xyz > 1e-9) & (case.xyz < 1 - 1e-9), axis=1)
    case.xyz = case.xyz.copy()
    case.xyz[inner] += np.random.default_rng(seed).uniform(-h, h, (int(inner.sum()), 3))
    return case


def relabelled(case):
    xyz, tets, dn, _ = eqsgen.permute_nodes(case.xyz, case.tets, case.dir_nodes, 7)
    order = np.argsort(dn, kind="stable")
    case.xyz, case.tets, case.dir_nodes, case.dir_drive = xyz, tets, dn[order].astype(np.int32), case.dir_drive[order]
    return case


def context(case, precision, **amg):
    c = Context(0, torch.cuda.current_stream(DEV))
    c.setup_case(case, precision=precision, **amg)
    return c


def solve(c, o, rhs, x0, classes=()):
    y = T(x0)
    c.profile_enable(classes)
    st = c.solve_M(T(rhs), y, RTOL)
    c.profile_enable(())
    x = y.cpu().numpy()
    res = np.linalg.norm(rhs - o.M_II @ x) / np.linalg.norm(rhs)
    assert res <= RTOL + 1e-14 * 10, res
    return st["iters"], x


SMALL = [
    ("c0 8", lambda: eqsgen.case_c0(8), EQS_PREC_FP64),           # operators in LDS
    ("c0 9", lambda: eqsgen.case_c0(9), EQS_PREC_FP32),
    ("c1 10", lambda: eqsgen.case_c1(n=10, seed=1), EQS_PREC_FP64),  # two rows a thread
    ("c1 11", lambda: eqsgen.case_c1(n=11, seed=1), EQS_PREC_FP32),
    ("c1 9 moved", lambda: moved(eqsgen.case_c1(n=9, seed=1)), EQS_PREC_FP64),
    ("c1 10 moved", lambda: moved(eqsgen.case_c1(n=10, seed=1)), EQS_PREC_FP32),
    ("c1 9 relabelled", lambda: relabelled(eqsgen.case_c1(n=9, seed=1)), EQS_PREC_FP64),
    ("p2 4", lambda: eqsgen.case_p2(4), EQS_PREC_FP64),
    ("p2 5", lambda: eqsgen.case_p2(5), EQS_PREC_FP32),
]


@pytest.mark.parametrize("name,maker,precision", SMALL, ids=[s[0] for s in SMALL])
def test_small_systems_in_one_launch(name, maker, precision, monkeypatch):
    case = maker()
    o = EqsOracle(case, dense_limit=0)
    rng = np.random.default_rng(3)
    xs = rng.standard_normal(o.n_free)
    rhs, x0 = o.M_II @ xs, 0.1 * rng.standard_normal(o.n_free)
    out = []
    for small in ("1", "0"):
        monkeypatch.setenv("EQS_SMALL", small)
        with context(case, precision) as c:
            assert ("one launch" in c.describe()) == (small == "1")
            it, x = solve(c, o, rhs, x0)
            zero = T(x0)
            assert c.solve_M(torch.zeros_like(zero), zero, RTOL)["iters"] == 0 and float(zero.abs().max()) == 0.0
            few = T(x0)
            st = c.solve_M(T(rhs), few, RTOL, maxit=3, allow_not_converged=True)
            assert st["iters"] == 3
            with pytest.raises(EqsError):
                c.solve_M(T(rhs), T(x0), RTOL, maxit=3)
            bad = rhs.copy()
            bad[5] = np.nan
            with pytest.raises(EqsError):
                c.solve_M(T(bad), T(x0), RTOL)
            again, x2 = solve(c, o, rhs, x0)  # nothing is left over from the failures
            assert again == it and np.array_equal(x, x2)
            out.append((it, few.cpu().numpy()))
    assert abs(out[0][0] - out[1][0]) <= 1
    # three iterations: the same Krylov vectors up to rounding (FP32 cycle: 2^-24 a term)
    tol = 1e-10 if precision == EQS_PREC_FP64 else 1e-5
    assert np.linalg.norm(out[0][1] - out[1][1]) <= tol * np.linalg.norm(out[0][1])


@pytest.mark.parametrize("precision", [EQS_PREC_FP64, EQS_PREC_FP32])
@pytest.mark.parametrize("maker,k", [(lambda: eqsgen.case_c1(n=23, seed=2), 3),
                                     (lambda: moved(eqsgen.case_c1(n=23, seed=2)), 7)])
def test_finest_matrices_by_diagonals(maker, k, precision, monkeypatch):
    case = maker()
    o = EqsOracle(case, dense_limit=0)
    rng = np.random.default_rng(4)
    rhs, x0 = o.M_II @ rng.standard_normal(o.n_free), np.zeros(o.n_free)
    out = []
    for dia in ("1", "0"):
        monkeypatch.setenv("EQS_DIAGONALS", dia)
        with context(case, precision) as c:
            assert (f"A0: {k} upper diagonals" in c.describe()) == (dia == "1")
            z = torch.zeros(o.n_free, dtype=torch.float64, device=DEV)
            c.apply_preconditioner(T(rhs), z)
            it, _ = solve(c, o, rhs, x0)
            out.append((it, z.cpu().numpy()))
    assert abs(out[0][0] - out[1][0]) <= 1
    tol = 1e-12 if precision == EQS_PREC_FP64 else 1e-5  # the cycle's own precision, 2^-53 and 2^-24 a term
    assert np.linalg.norm(out[0][1] - out[1][1]) <= tol * np.linalg.norm(out[0][1])


def test_batch_by_diagonals_keeps_instances_apart(monkeypatch):
    """Uneven instances, one of them with other diagonals; a state that is not a
    number stops its own instance only."""
    cases = [eqsgen.case_c1(n=9, seed=1), moved(eqsgen.case_c1(n=8, seed=2)), eqsgen.case_c1(n=11, seed=3)]
    outs = []
    for dia in ("1", "0"):
        monkeypatch.setenv("EQS_DIAGONALS", dia)
        inputs = []
        for c in cases:
            ctx = Context(0, torch.cuda.current_stream(DEV))
            ctx.set_inputs(c)
            inputs.append(ctx)
        b = Batch(inputs, precision=EQS_PREC_FP64, stream=torch.cuda.current_stream(DEV))
        xs = [torch.zeros(c.n_nodes, dtype=torch.float64, device=DEV) for c in cases]
        b.rkc_steps(2, 0.0, 1e-4, 8, xs, 1e-12)
        outs.append([x.cpu().numpy() for x in xs])
        xs[0][:] = float("nan")
        try:
            b.rkc_steps(1, 2e-4, 1e-4, 8, xs, 1e-12)
        except EqsError:
            pass
        assert all(bool(torch.isfinite(x).all()) for x in xs[1:])
        b.close()
        for ctx in inputs:
            ctx.close()
    for p, q in zip(*outs):
        assert np.linalg.norm(p - q) <= 1e-9 * np.linalg.norm(p)  # two solutions to 1e-12 with condition numbers below 1e3


@pytest.mark.parametrize("n", [20, 45, 47, 72])
def test_reductions_by_the_next_kernel_or_by_finalisers(n):
    """n = 45 and 47 lie on either side of 100,000 rows; n = 72 has more row
    blocks (1,498) than the kernels' workgroups of one row a thread."""
    case = eqsgen.case_c1(n=n, seed=1)
    o = EqsOracle(case, dense_limit=0)
    rng = np.random.default_rng(5)
    rhs, x0 = o.M_II @ rng.standard_normal(o.n_free), 0.1 * rng.standard_normal(o.n_free)
    with context(case, EQS_PREC_FP32) as c:
        its = [solve(c, o, rhs, x0, classes)[0] for classes in ((), ("finalise",), ("spmv_M",))]
    assert max(its) - min(its) <= 1, its


@pytest.mark.parametrize("precision", [EQS_PREC_FP64, EQS_PREC_FP32])
def test_columns_from_a_base_per_pair(precision, monkeypatch):
    """[G Q] on level 1 of 61^3 cells, whose columns 33,000 rows apart fit no offset
    from the row: from pairs' bases, in every number of lanes a row, and as 32-bit
    columns (EQS_INDEX16=0). The same entries in the same lanes, so sums differ by
    their order only where the two parts of a row begin at a pair of their own."""
    case = eqsgen.case_c1(n=61, seed=1)
    z = []
    rng = np.random.default_rng(6)
    for layout, index16 in [("1", "1"), ("2", "1"), ("4", "1"), ("8", "1"), ("1", "0"), ("4", "0")]:
        monkeypatch.setenv("EQS_LAYOUT", "sell" + layout)
        monkeypatch.setenv("EQS_INDEX16", index16)
        with context(case, precision) as c:
            n = c.info()["n_free"]
            if not z:
                r = rng.standard_normal(n)
            out = torch.zeros(n, dtype=torch.float64, device=DEV)
            c.apply_preconditioner(T(r), out)
            z.append(out.cpu().numpy())
    tol = 1e-13 if precision == EQS_PREC_FP64 else 2e-6  # some 50 terms of 2^-53, 2^-24 each
    for v in z[1:]:
        assert np.linalg.norm(v - z[0]) <= tol * np.linalg.norm(z[0])


@pytest.mark.parametrize("graph_iters", [1, 3])
@pytest.mark.parametrize("n", [8, 23, 47])
def test_captured_iterations_match_plain_launches(n, graph_iters):
    """On a stream of its own a context replays captured iterations; on the null
    stream it launches them one by one. Several solves in a row, each against the
    true residual, and steps in between."""
    case = eqsgen.case_c1(n=n, seed=1)
    o = EqsOracle(case, dense_limit=0)
    rng = np.random.default_rng(8)
    rhs = [o.M_II @ rng.standard_normal(o.n_free) for _ in range(3)]
    out = []
    for stream in (torch.cuda.current_stream(DEV), torch.cuda.Stream(DEV)):
        with torch.cuda.stream(stream):
            c = Context(0, stream)
            c.setup_case(case, precision=EQS_PREC_FP32)
            c.set_graph_iters(graph_iters)
            x = torch.zeros(case.n_nodes, dtype=torch.float64, device=DEV)
            its = []
            for k, b in enumerate(rhs):
                its.append(solve(c, o, b, np.zeros(o.n_free))[0])
                c.rkc_step(k * case.tau, case.tau, 8, x, 1e-12)
            stream.synchronize()
            out.append((its, x.cpu().numpy()))
            c.close()
    assert max(abs(p - q) for p, q in zip(out[0][0], out[1][0])) <= 1
    assert np.linalg.norm(out[0][1] - out[1][1]) <= 1e-9 * np.linalg.norm(out[0][1])
