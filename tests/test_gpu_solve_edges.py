"""CG solves on M that need no iteration, in every form of the iteration: one or
several iterations per launch, launched one by one (null stream) or captured
(a stream of its own), reductions by the next kernel or by finaliser launches
(timing the finaliser class asks for those); a single system too large for the
one-launch solve, and two instances in one context.

A right-hand side of zero gives zero whatever the start vector and whatever was
solved before; a start vector that already meets the tolerance stays as it is,
also in a context's first solve and with no iterations allowed. Both are exact
statements, so the comparisons are exact. The ordinary solves between them are
checked by |b - M x| <= rtol |b|, with 1e-13 for the rounding of the check's own
product (15 terms of relative 2^-53, |M||x| within 1e1 of |b|).
"""

import numpy as np
import pytest

import eqsgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1612_09447_amd import EQS_PREC_FP32, EQS_PREC_FP64, Context  # noqa: E402

DEV = torch.device("cuda:0")
RTOL = 1e-11


def single(stream, precision):
    c = Context(0, stream)
    c.setup_case(eqsgen.case_c1(n=14, seed=1), precision=precision)
    return c, [0, c.info()["n_free"]]


def two_instances(stream, precision):
    """The second instance begins inside a 256-row block of the first one."""
    cases = [eqsgen.case_c1(n=9, seed=1), eqsgen.case_c1(n=8, seed=2)]
    c = Context(0, stream)
    nodes, tets, rows = [0], [0], [0]
    for k in cases:
        nodes.append(nodes[-1] + k.n_nodes)
        tets.append(tets[-1] + len(k.tets))
        rows.append(rows[-1] + k.n_nodes - len(k.dir_nodes))
    assert rows[1] % 256 != 0
    c.set_mesh(np.concatenate([k.xyz for k in cases]),
               np.concatenate([k.tets + o for k, o in zip(cases, nodes)]).astype(np.int32))
    c.set_instances(np.array(nodes, dtype=np.int64), np.array(tets, dtype=np.int64))
    mats, drives = np.cumsum([0] + [k.n_mat for k in cases]), np.cumsum([0] + [len(k.amp) for k in cases])
    join = lambda name: np.concatenate([getattr(k, name) for k in cases])  # noqa: E731
    c.set_materials(*(join(a) for a in ("eps_r", "kappa0", "e_s", "alpha", "nonlinear")),
                    np.concatenate([k.tet_mat + o for k, o in zip(cases, mats)]))
    c.set_dirichlet(np.concatenate([k.dir_nodes + o for k, o in zip(cases, nodes)]),
                    np.concatenate([k.dir_drive + o for k, o in zip(cases, drives)]),
                    *(join(a) for a in ("amp", "freq", "phase")))
    c.build_preconditioner(precision=precision)
    return c, rows


@pytest.mark.parametrize("classes", [(), ("finalise",)], ids=["sums by consumers", "finalisers"])
@pytest.mark.parametrize("own_stream", [False, True], ids=["launched", "captured"])
@pytest.mark.parametrize("graph_iters", [1, 2, 5])
@pytest.mark.parametrize("make,precision", [(single, EQS_PREC_FP32), (single, EQS_PREC_FP64),
                                            (two_instances, EQS_PREC_FP64)])
def test_solves_without_an_iteration(make, precision, graph_iters, own_stream, classes):
    stream = torch.cuda.Stream(DEV) if own_stream else torch.cuda.current_stream(DEV)
    with torch.cuda.stream(stream):
        c, rows = make(stream, precision)
        with c:
            assert "one launch" not in c.describe()
            c.set_graph_iters(graph_iters)
            c.profile_enable(classes)
            n = rows[-1]
            rng = np.random.default_rng(9)
            xs = torch.as_tensor(rng.standard_normal(n), device=DEV)
            rhs, zero = torch.empty_like(xs), torch.zeros_like(xs)
            c.apply_M(xs, rhs)
            for maxit in (100, 0):  # the context's first solve: nothing to do
                y = xs.clone()
                st = c.solve_M(rhs, y, RTOL, maxit=maxit)
                assert st["iters"] == 0 and torch.equal(y, xs)
            for _ in range(2):
                y = 0.1 * xs
                assert c.solve_M(rhs, y, RTOL)["iters"] > 0
                r = torch.empty_like(y)
                c.apply_M(y, r)
                res = float(torch.linalg.vector_norm(rhs - r) / torch.linalg.vector_norm(rhs))
                assert res <= RTOL + 1e-13, res
                y = xs.clone()
                st = c.solve_M(zero, y, RTOL)
                assert st["iters"] == 0 and torch.equal(y, zero)
                y = xs.clone()  # and after a solve with a right-hand side of zero
                st = c.solve_M(rhs, y, RTOL)
                assert st["iters"] == 0 and torch.equal(y, xs)
            for i in range(len(rows) - 1 if len(rows) > 2 else 0):  # one instance's share of it is zero
                part = rhs.clone()
                part[rows[i]:rows[i + 1]] = 0.0
                y = 0.1 * xs
                c.solve_M(part, y, RTOL)
                assert not bool(y[rows[i]:rows[i + 1]].any())
                c.apply_M(y, r)
                for k in range(len(rows) - 1):
                    a, b = rows[k], rows[k + 1]
                    assert float(torch.linalg.vector_norm((part - r)[a:b])) <= (RTOL + 1e-13) * float(
                        torch.linalg.vector_norm(part[a:b]))
            stream.synchronize()


@pytest.mark.parametrize("n", [68, 69, 83, 84])
def test_plain_cycle_on_many_row_blocks(n, monkeypatch):
    """The plain cycle takes one row per thread whatever the size: 1,247, 1,302, 2,261
    and 2,343 row blocks, on both sides of the counts up to which the next kernel
    sums them (1,281 and 2,305). Solved to the true residual, in as many iterations
    as with finaliser launches, up to the one that rounding can cost."""
    monkeypatch.setenv("EQS_FOLD", "0")
    monkeypatch.setenv("EQS_AUTOTUNE", "0")
    with Context(0, torch.cuda.current_stream(DEV)) as c:
        c.setup_case(eqsgen.case_c1(n=n, seed=1), precision=EQS_PREC_FP32)
        rng = np.random.default_rng(10)
        xs = torch.as_tensor(rng.standard_normal(c.info()["n_free"]), device=DEV)
        rhs, r, its = torch.empty_like(xs), torch.empty_like(xs), []
        c.apply_M(xs, rhs)
        for classes in ((), ("finalise",)):
            y = torch.zeros_like(xs)
            c.profile_enable(classes)
            its.append(c.solve_M(rhs, y, RTOL, maxit=200)["iters"])
            c.profile_enable(())
            c.apply_M(y, r)
            res = float(torch.linalg.vector_norm(rhs - r) / torch.linalg.vector_norm(rhs))
            assert res <= RTOL + 1e-13, res
    assert abs(its[0] - its[1]) <= 1, its
