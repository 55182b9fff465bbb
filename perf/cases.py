"""Performance cases of the explicit-RKC library: the work its users have it do,
through its public entry points, over the sizes and options of the repository's
workloads (eqsgen/configs), tests and benchmark.

Kinds of case (``op``):
  step      one RKC(s) step of one instance (Context.rkc_step): the time loop's
            body; every pass is the next step of the run, so the start vectors
            are those of a run
  batch     one RKC(s) step of several independent, uneven instances (Batch)
  rhs       one stage right-hand side b(t) - K(x)x (Context.stage_rhs)
  solve     one solve with M from a zero start vector (Context.solve_M)
  galerkin  the start vector of eq. (5) from a window the caller holds
            (Context.galerkin_start)
  mlp       the start-vector network's online training of one stage (its pairs
            in minibatches of up to 64, one Adam step each) and a prediction
            for every pair (Mlp.train_step, Mlp.forward, Mlp.get)

A context is set up once per mesh and kept, as a program keeps it. A run's own
state inside a context (the last stage solution) is taken back to "none" when a
case is prepared; cases with an estimator start vector, whose window holds the
run's solutions, have a context of their own per run.

``exact`` gives the same results from the definitions in plain torch, in 64
bits: element-by-element K(x)x, an assembled M, Jacobi-preconditioned CG to
1e-13, the RKC recurrence, eq. (5) by dense solves, the network by matrix
products.
"""

import math

import numpy as np
import torch

import eqsgen
from paper_1612_09447_amd import EQS_PREC_FP32, EQS_PREC_FP64, Batch, Context, Mlp

DEV = "cuda"
EPS0 = 8.8541878128e-12
TAU = 1e-4  # every workload's step
# Steps solve to 1e-10 (c0's tolerance) or 1e-12 (the paper's and the smoke run's): the workloads' loosest, 1e-8,
# leaves the potentials open in the ninth digit, where two correct runs differ.


def listed():
    return [
        # the smallest mesh in use: the slab problem of the c0 configuration, where a step is all launches and waits
        {"name": "step_c0", "op": "step", "recipe": "c0", "n": 8, "s": 8, "precision": "fp64", "rtol": 1e-10,
         "guess": "previous", "relabel": False},
        # one of the batched workload's instances on its own, with its nodes numbered in no order, as mesh files
        # that are not structured come
        {"name": "step_unordered", "op": "step", "recipe": "c1", "n": 40, "s": 8, "precision": "fp32", "rtol": 1e-10,
         "guess": "previous", "relabel": True},
        # the c1 configuration: 266,175 free nodes, all in 64 bits
        {"name": "step_c1", "op": "step", "recipe": "c1", "n": 64, "s": 12, "precision": "fp64", "rtol": 1e-10,
         "guess": "previous", "relabel": False},
        # the c2 configuration, the benchmark's: 2,113,407 free nodes, 32-bit hierarchy under 64-bit CG
        {"name": "step_c2", "op": "step", "recipe": "c1", "n": 128, "s": 16, "precision": "fp32", "rtol": 1e-10,
         "guess": "previous", "relabel": False},
        # the learned start vector (c4 configuration) on a mid-size mesh
        {"name": "step_learned", "op": "step", "recipe": "c1", "n": 64, "s": 16, "precision": "fp32", "rtol": 1e-10,
         "guess": "mlp", "relabel": False},
        # eq. (5)'s start vector inside a run, odd size
        {"name": "step_galerkin", "op": "step", "recipe": "c1", "n": 51, "s": 16, "precision": "fp32", "rtol": 1e-10,
         "guess": "galerkin", "relabel": False},
        # second-order (10-node) tets: the p2 configuration's recipe, 270,465 free nodes
        {"name": "step_p2", "op": "step", "recipe": "p2", "n": 32, "s": 16, "precision": "fp32", "rtol": 1e-10,
         "guess": "previous", "relabel": False},
        # uneven instances of the c3 configuration in one batch
        {"name": "batch_c3", "op": "batch", "instances": 12, "base_seed": 3000, "s": 8, "precision": "fp32",
         "rtol": 1e-10},
        # the fused element pass alone at the benchmark's size: the paper's "K assembly" time
        {"name": "rhs_c2", "op": "rhs", "recipe": "c1", "n": 128, "order": 1},
        # the linear solver alone, at the paper's tolerance of 1e-12, between the two large configurations
        {"name": "solve_96", "op": "solve", "recipe": "c1", "n": 96, "precision": "fp32", "rtol": 1e-12},
        # eq. (5) on a full window at the benchmark's size
        {"name": "galerkin_c2", "op": "galerkin", "n": 128, "k": 16},
        # a stage's training of the network: 256 pairs, four minibatches
        {"name": "mlp_stage", "op": "mlp", "pairs": 256, "bf16": True},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("step", "step", "step", "guess", "p2", "batch", "rhs", "solve", "galerkin", "mlp"))
    prec = rng.choice(("fp64", "fp32"))
    if op == "step":
        n = _log_int(rng, 6, 112)
        return {"op": "step", "recipe": rng.choice(("c0", "c1", "c1")), "n": n, "s": rng.choice((8, 12, 16)),
                "precision": prec, "rtol": rng.choice((1e-10, 1e-12)), "guess": "previous",
                "relabel": n <= 48 and rng.random() < 0.25}
    if op == "guess":
        return {"op": "step", "recipe": "c1", "n": _log_int(rng, 24, 64), "s": rng.choice((12, 16)),
                "precision": prec, "rtol": 1e-10, "guess": rng.choice(("galerkin", "mlp")), "relabel": False}
    if op == "p2":
        return {"op": "step", "recipe": "p2", "n": _log_int(rng, 5, 32), "s": rng.choice((8, 16)),
                "precision": prec, "rtol": 1e-10, "guess": "previous", "relabel": False}
    if op == "batch":
        return {"op": "batch", "instances": rng.randint(3, 12), "base_seed": 3000 + rng.randint(0, 60),
                "s": 8, "precision": "fp32", "rtol": 1e-10}
    if op == "rhs":
        order = rng.choice((1, 1, 2))
        return {"op": "rhs", "recipe": "c1" if order == 1 else "p2",
                "n": _log_int(rng, 8, 112 if order == 1 else 40), "order": order}
    if op == "solve":
        return {"op": "solve", "recipe": "c1", "n": _log_int(rng, 8, 96), "precision": prec, "rtol": 1e-12}
    if op == "galerkin":
        return {"op": "galerkin", "n": _log_int(rng, 16, 112), "k": rng.randint(2, 16)}
    return {"op": "mlp", "pairs": rng.randint(16, 256), "bf16": rng.random() < 0.7}


# ------------------------------------------------------------------ inputs
_meshes, _contexts, _idle = {}, {}, {}


def _mesh(recipe, n, relabel=False):
    """The workload's mesh, materials and Dirichlet data (a function of the arguments)."""
    key = (recipe, n, relabel)
    if key not in _meshes:
        if len(_meshes) > 6:
            _meshes.clear()
        c = {"c0": eqsgen.case_c0, "c1": eqsgen.case_c1, "p2": eqsgen.case_p2}[recipe](n)
        if relabel:
            xyz, tets, dn, perm = eqsgen.permute_nodes(c.xyz, c.tets, c.dir_nodes, 7)
            order = np.argsort(dn, kind="stable")
            c.xyz, c.tets, c.dir_nodes, c.dir_drive = xyz, tets, dn[order].astype(np.int32), c.dir_drive[order]
        _meshes[key] = c
    return _meshes[key]


def _precision(name):
    return EQS_PREC_FP32 if name == "fp32" else EQS_PREC_FP64


def _context(recipe, n, precision, relabel=False):
    """The context of a mesh, set up once, and what takes its run state back to none."""
    key = (recipe, n, precision, relabel)
    if key not in _contexts:
        ctx = Context(0, torch.cuda.current_stream())
        ctx.setup_case(_mesh(recipe, n, relabel), precision=_precision(precision))
        _contexts[key] = (ctx, ctx.state_save())
    ctx, none = _contexts[key]
    ctx.state_load(none)
    return ctx


class _Own:
    """A context that one run has to itself; it goes back for the next run when this one is dropped."""

    def __init__(self, case):
        key = (case["recipe"], case["n"], case["precision"])
        self.free = _idle.setdefault(key, [])
        if self.free:
            self.ctx, self.none = self.free.pop()
        else:
            self.ctx = Context(0, torch.cuda.current_stream())
            self.ctx.setup_case(_mesh(case["recipe"], case["n"]), precision=_precision(case["precision"]))
            self.ctx.set_guess("previous")
            self.none = self.ctx.state_save()
        self.ctx.set_guess("previous")
        self.ctx.state_load(self.none)

    def __del__(self):
        self.free.append((self.ctx, self.none))


def _start(mesh, seed, offset=0):
    """(t, x): a state that a run meets in the first part of its drive's period (before the varistors switch, so
    that the linear profile of the drive's value is near it), with smooth deviations of a few per cent. A run
    goes on from there through the switching."""
    t = float(np.random.default_rng(seed).uniform(1e-4, 4e-4))
    r = np.random.default_rng(seed + offset)
    xyz = torch.as_tensor(mesh.xyz, device=DEV)
    amp = float(mesh.amp[1]) * math.sin(2 * math.pi * float(mesh.freq[1]) * t)
    x = xyz[:, 2] * amp
    for _ in range(6):
        a, kx, ky, kz = r.uniform(-0.02, 0.02), r.integers(0, 4), r.integers(0, 4), r.integers(1, 4)
        x = x + (amp * a) * torch.cos(math.pi * kx * xyz[:, 0]) * torch.cos(math.pi * ky * xyz[:, 1]) * torch.sin(
            math.pi * kz * xyz[:, 2])
    return t, x.contiguous()


def _batch_cases(case):
    key = ("batch", case["instances"], case["base_seed"])
    if key not in _meshes:
        _meshes[key] = eqsgen.case_batch(case["instances"], case["base_seed"])
    return _meshes[key]


def _batch_start(case, seed):
    starts = [_start(c, seed, 1000 * i) for i, c in enumerate(_batch_cases(case))]
    return starts[0][0], [x for _, x in starts]


def _window(nf, k, seed):
    """k columns like a window of stage solutions: one profile that changes little from
    column to column, with differences down to a thousandth of it; and a right-hand side's
    solution near them."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    base = torch.randn(nf, generator=g, device=DEV, dtype=torch.float64)
    S = torch.empty(k, nf, device=DEV, dtype=torch.float64)
    for a in range(k):
        S[a] = base * (1.0 + 0.02 * a) + torch.randn(nf, generator=g, device=DEV, dtype=torch.float64) * (
            10.0 ** (-3.0 * a / max(1, k - 1)))
    return S, 0.5 * S[0] + base * 0.3 + 0.01 * torch.randn(nf, generator=g, device=DEV, dtype=torch.float64)


def _pairs(case, seed):
    """Training pairs as the estimator forms them: two unit vectors in, targets of order one."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(case["pairs"], 2, 16, generator=g, device=DEV)
    x = (x / x.norm(dim=2, keepdim=True)).reshape(case["pairs"], 32).contiguous()
    w = torch.randn(32, 16, generator=g, device=DEV) * 0.3
    return x, (x @ w + 0.05 * torch.randn(case["pairs"], 16, generator=g, device=DEV)).contiguous()


def prepare(case, seed):
    op = case["op"]
    if op == "step":
        mesh = _mesh(case["recipe"], case["n"], case["relabel"])
        own = _Own(case) if case["guess"] != "previous" else None
        ctx = own.ctx if own else _context(case["recipe"], case["n"], case["precision"], case["relabel"])
        if own:
            ctx.set_guess(case["guess"], init=eqsgen.mlp_init(4) if case["guess"] == "mlp" else None)
        t, x = _start(mesh, seed)
        return {"op": op, "ctx": ctx, "own": own, "t": t, "x": x, "s": case["s"], "rtol": case["rtol"]}
    if op == "batch":
        key = ("batch", case["instances"], case["base_seed"], case["precision"])
        if key not in _contexts:
            ctxs = []
            for c in _batch_cases(case):
                ctx = Context(0, torch.cuda.current_stream())
                ctx.set_inputs(c)
                ctxs.append(ctx)
            _contexts[key] = Batch(ctxs, precision=_precision(case["precision"]), stream=torch.cuda.current_stream())
        t, xs = _batch_start(case, seed)
        return {"op": op, "batch": _contexts[key], "xs": xs, "t": t, "s": case["s"], "rtol": case["rtol"]}
    if op == "rhs":
        mesh = _mesh(case["recipe"], case["n"])
        ctx = _context(case["recipe"], case["n"], "fp32")
        t, x = _start(mesh, seed)
        y = x[_free(mesh)].contiguous()
        return {"op": op, "ctx": ctx, "t": t, "y": y, "r": torch.empty_like(y)}
    if op == "solve":
        mesh = _mesh(case["recipe"], case["n"])
        ctx = _context(case["recipe"], case["n"], case["precision"])
        t, x = _start(mesh, seed)
        rhs = _Plain(mesh, matrix=False).rhs(t, x).contiguous()
        return {"op": op, "ctx": ctx, "rhs": rhs, "y": torch.empty_like(rhs), "rtol": case["rtol"]}
    if op == "galerkin":
        ctx = _context("c1", case["n"], "fp32")
        S, f = _window(ctx.info()["n_free"], case["k"], seed)
        R, r = torch.empty_like(S), torch.empty_like(f)
        for a in range(case["k"]):
            ctx.apply_M(S[a], R[a])
        ctx.apply_M(f, r)
        return {"op": op, "ctx": ctx, "S": S, "R": R, "r": r, "x0": torch.empty_like(r)}
    if op == "mlp":
        x, t = _pairs(case, seed)
        net = Mlp(eqsgen.mlp_init(seed), bf16=case["bf16"], stream=torch.cuda.current_stream())
        return {"op": op, "net": net, "x": x, "t": t, "y": torch.empty(case["pairs"], 16, device=DEV)}
    raise ValueError(op)


def run(state):
    op = state["op"]
    if op == "step":
        state["ctx"].rkc_step(state["t"], TAU, state["s"], state["x"], state["rtol"])
        state["t"] += TAU
        return state["x"]
    if op == "batch":
        state["batch"].rkc_steps(1, state["t"], TAU, state["s"], state["xs"], state["rtol"])
        state["t"] += TAU
        return state["xs"]
    if op == "rhs":
        state["ctx"].stage_rhs(state["t"], state["y"], state["r"])
        return state["r"]
    if op == "solve":
        state["y"].zero_()
        state["ctx"].solve_M(state["rhs"], state["y"], state["rtol"])
        return state["y"]
    if op == "galerkin":
        m = state["ctx"].galerkin_start(state["S"], state["R"], state["r"], state["x0"])
        return {"x0": state["x0"], "kept": m}
    if op == "mlp":
        net, x, t = state["net"], state["x"], state["t"]
        losses = [net.train_step(x[b:b + 64], t[b:b + 64]) for b in range(0, x.shape[0], 64)]
        net.forward(x, state["y"])
        params, grads = net.get()
        return {"loss": losses, "y": state["y"], "params": params, "grads": grads}
    raise ValueError(op)


# -------------------------------------------------------------------- work
def _counts(recipe, n):
    """(tets, nodes, free nodes, nonzeros of M) of a Kuhn mesh, closed form: first-order M is the 7-point
    stencil; a second-order row holds 23 entries on average."""
    m = n + 1 if recipe != "p2" else 2 * n + 1
    free = m * m * (m - 2)
    return 6 * n ** 3, m ** 3, free, (7 if recipe != "p2" else 23) * free


def _pass_work(recipe, n):
    """An element pass: connectivity, material and (per node) coordinates, potential, result."""
    tets, nodes, _, _ = _counts(recipe, n)
    per = (16, 150) if recipe != "p2" else (40, 900)
    return tets * (per[0] + 4) + nodes * 40, tets * per[1]


def _solve_work(recipe, n, iters):
    """CG iterations: M's values once each (half of a symmetric matrix), x, r, p, q, z."""
    _, _, free, nnz = _counts(recipe, n)
    return iters * (nnz / 2 * 8 + 9 * 8 * free), iters * (4 * nnz + 12 * free)


def work(case):
    op = case["op"]
    if op == "mlp":
        steps = case["pairs"]
        return {"bytes": 4 * (48 + 16) * steps + 4 * 7312 * 8, "flops": steps * 7168 * 2 * 4}
    if op == "galerkin":
        _, _, free, _ = _counts("c1", case["n"])
        k = case["k"]
        return {"bytes": 8 * free * (2 * k + 2), "flops": 2 * free * (2 * k * k + 2 * k)}
    if op == "batch":
        tot = [0.0, 0.0]
        for i in range(case["instances"]):
            n = int(np.random.default_rng(case["base_seed"] + i).choice((16, 24, 32, 40, 48)))
            for k, v in enumerate(_step_work("c1", n, case["s"], 4)):
                tot[k] += v
        return {"bytes": tot[0], "flops": tot[1]}
    if op == "rhs":
        b, f = _pass_work(case["recipe"], case["n"])
    elif op == "solve":
        b, f = _solve_work(case["recipe"], case["n"], 12)
    else:
        b, f = _step_work(case["recipe"], case["n"], case["s"], 4)
    return {"bytes": b, "flops": f}


def _step_work(recipe, n, s, iters):
    """s stages of an element pass, a solve (few iterations even from a good start) and the combination."""
    pb, pf = _pass_work(recipe, n)
    sb, sf = _solve_work(recipe, n, iters)
    free = _counts(recipe, n)[2]
    return s * (pb + sb + 6 * 8 * free), s * (pf + sf + 9 * free)


# ------------------------------------------- the same in plain torch, 64 bits
def _free(mesh):
    mask = torch.ones(mesh.n_nodes, dtype=torch.bool, device=DEV)
    mask[torch.as_tensor(mesh.dir_nodes, device=DEV).long()] = False
    return torch.nonzero(mask).reshape(-1)


class _Plain:
    """M and K(x)x of a mesh from the element definitions (4- or 10-node tets)."""

    EDGES = ((0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3))
    CHUNK = 1 << 20

    def __init__(self, mesh, matrix=True):
        f64 = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=DEV)  # noqa: E731
        self.xyz = f64(mesh.xyz)
        self.tets = torch.as_tensor(mesh.tets, device=DEV)
        self.mat = torch.as_tensor(mesh.tet_mat, device=DEV).long()
        self.eps, self.k0, self.es, self.al = EPS0 * f64(mesh.eps_r), f64(mesh.kappa0), f64(mesh.e_s), f64(mesh.alpha)
        self.nl = torch.as_tensor(np.asarray(mesh.nonlinear), device=DEV) != 0
        self.dn = torch.as_tensor(mesh.dir_nodes, device=DEV).long()
        dd = np.asarray(mesh.dir_drive)
        self.amp, self.om, self.ph = f64(mesh.amp[dd]), f64(2 * math.pi * mesh.freq[dd]), f64(mesh.phase[dd])
        self.free = _free(mesh)
        self.n_nodes = mesh.n_nodes
        if self.tets.shape[1] == 10:  # the 4-point rule of degree 2
            a, b = (5 + 3 * math.sqrt(5)) / 20, (5 - math.sqrt(5)) / 20
            self.points = [[a if q == v else b for v in range(4)] for q in range(4)]
        else:
            self.points = None
        if matrix:
            self._assemble()

    def _cofactors(self, tets):
        p = self.xyz[tets[:, :4].long()]
        e1, e2, e3 = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0], p[:, 3] - p[:, 0]
        c1, c2, c3 = torch.linalg.cross(e2, e3), torch.linalg.cross(e3, e1), torch.linalg.cross(e1, e2)
        return torch.stack([-(c1 + c2 + c3), c1, c2, c3], 1), (e1 * c1).sum(1).abs()

    def _shape_gradients(self, cof):
        """Per quadrature point the scaled gradients of the element's shape functions."""
        if self.points is None:
            return [cof]
        out = []
        for lam in self.points:
            g = [(4 * lam[v] - 1) * cof[:, v] for v in range(4)]
            g += [4 * (lam[b] * cof[:, a] + lam[a] * cof[:, b]) for a, b in self.EDGES]
            out.append(torch.stack(g, 1))
        return out

    def _chunks(self):
        for a in range(0, self.tets.shape[0], self.CHUNK):
            yield self.tets[a:a + self.CHUNK], self.mat[a:a + self.CHUNK]

    def _assemble(self):
        nf = self.free.numel()
        where = torch.full((self.n_nodes,), -1, dtype=torch.long, device=DEV)
        where[self.free] = torch.arange(nf, device=DEV)
        keys, vals = None, None
        for tets, mat in self._chunks():
            cof, det = self._cofactors(tets)
            grads = self._shape_gradients(cof)
            el = sum(g @ g.transpose(1, 2).contiguous() for g in grads)
            el = el * (self.eps[mat] / (6 * len(grads) * det))[:, None, None]
            loc = where[tets.long()]
            i, j = loc[:, :, None].expand_as(el), loc[:, None, :].expand_as(el)
            keep = (i >= 0) & (j >= 0)
            k, v = (i * nf + j)[keep], el[keep]
            if keys is not None:
                k, v = torch.cat([keys, k]), torch.cat([vals, v])
            keys, inv = torch.unique(k, return_inverse=True)
            vals = torch.zeros(keys.numel(), dtype=torch.float64, device=DEV).index_add_(0, inv, v)
        rows = keys // nf
        cols = keys - rows * nf
        self.diag = vals[rows == cols]
        keep = vals.abs() > 1e-14 * (self.diag[rows] * self.diag[cols]).sqrt()  # exact zeros up to round-off
        rows, cols, vals = rows[keep], cols[keep], vals[keep]
        count = torch.bincount(rows, minlength=nf)
        place = torch.arange(rows.numel(), device=DEV) - (torch.cumsum(count, 0) - count)[rows]
        width = int(count.max())  # every row padded to the longest, entry by entry
        self.cols = torch.zeros(width, nf, dtype=torch.int32, device=DEV)
        self.vals = torch.zeros(width, nf, dtype=torch.float64, device=DEV)
        self.cols[place, rows], self.vals[place, rows] = cols.int(), vals

    def mul(self, x):
        y = self.vals[0] * x[self.cols[0]]
        for c, v in zip(self.cols[1:], self.vals[1:]):
            y.addcmul_(v, x[c])
        return y

    def boundary(self, t):
        """The Dirichlet values and rates at t."""
        w = self.om * t + self.ph
        return self.amp * torch.sin(w), self.om * self.amp * torch.cos(w)

    def rhs(self, t, x):
        """b(t) - [K(x)x] on the free nodes; x on all nodes, its Dirichlet entries taken from the drives."""
        g, rate = self.boundary(t)
        u, v = x.clone(), torch.zeros_like(x)
        u[self.dn], v[self.dn] = g, rate
        out = torch.zeros_like(u)
        for tets, mat in self._chunks():
            cof, det = self._cofactors(tets)
            ids = tets.long()
            ue, ve = u[ids], v[ids]
            grads = self._shape_gradients(cof)
            y = 0.0
            for gr in grads:
                w = (gr * ue[:, :, None]).sum(1)
                field = w.norm(dim=1) / det
                kap = self.k0[mat] * (1 + torch.where(self.nl[mat], (field / self.es[mat]) ** self.al[mat], 0.0))
                w = kap[:, None] * w + self.eps[mat][:, None] * (gr * ve[:, :, None]).sum(1)
                y = y + (gr * w[:, None, :]).sum(2)
            out.index_add_(0, ids.reshape(-1), (y / (6 * len(grads) * det)[:, None]).reshape(-1))
        return -out[self.free]

    def solve(self, b, x, rtol=1e-13):
        """M x = b by Jacobi-preconditioned CG from x."""
        x = x.clone()
        inv = 1.0 / self.diag
        bb = torch.dot(b, b)
        for _ in range(3):  # from the true residual
            r = b - self.mul(x)
            if not bool(torch.dot(r, r) > rtol * rtol * bb):
                break
            z = inv * r
            p, rz = z.clone(), torch.dot(r, z)
            for it in range(6000):
                q = self.mul(p)
                a = rz / torch.dot(p, q)
                x += a * p
                r -= a * q
                z = inv * r
                rz, old = torch.dot(r, z), rz
                p = z + (rz / old) * p
                if it % 25 == 24 and not bool(torch.dot(r, r) > rtol * rtol * bb):
                    break
        return x

    def step(self, t, dt, s, x):
        """One RKC(s) step (second order, damping 2/13) from x, all nodes."""
        w0 = 1 + (2 / 13) / s ** 2
        T, D, E = [1.0, w0], [0.0, 1.0], [0.0, 0.0]
        for j in range(2, s + 1):
            T.append(2 * w0 * T[-1] - T[-2])
            D.append(2 * T[j - 1] + 2 * w0 * D[-1] - D[-2])
            E.append(4 * D[j - 1] + 2 * w0 * E[-1] - E[-2])
        w1 = D[s] / E[s]
        b = [0.0, 0.0] + [E[j] / D[j] ** 2 for j in range(2, s + 1)]
        b[0] = b[1] = b[2]
        c = [0.0, b[1] * w1] + [w1 * E[j] / D[j] for j in range(2, s + 1)]
        full = x.clone()

        def slope(tj, y, start):
            full[self.free] = y
            return self.solve(self.rhs(tj, full), start)

        y0 = x[self.free]
        f0 = slope(t, y0, torch.zeros_like(y0))
        ym, y, f = y0, y0 + b[1] * w1 * dt * f0, f0
        for j in range(2, s + 1):
            f = slope(t + c[j - 1] * dt, y, f)
            mu, nu, mt = 2 * b[j] * w0 / b[j - 1], -b[j] / b[j - 2], 2 * b[j] * w1 / b[j - 1]
            ga = -(1 - b[j - 1] * T[j - 1]) * mt
            ym, y = y, (1 - mu - nu) * y0 + mu * y + nu * ym + mt * dt * f + ga * dt * f0
        out = x.clone()
        out[self.free] = y
        out[self.dn] = self.boundary(t + dt)[0]
        return out


def _plain_network(case, seed):
    """The training steps and the prediction in 64 bits; operands rounded to bfloat16 where the network rounds them."""
    x, t = (v.double() for v in _pairs(case, seed))
    q = (lambda v: v.float().bfloat16().double()) if case["bf16"] else (lambda v: v)
    names = ("W1", "b1", "W2", "b2", "W3", "b3")
    init = eqsgen.mlp_init(seed)
    p = {k: torch.as_tensor(init[k], device=DEV).double() for k in names}
    m, v = ({k: torch.zeros_like(p[k]) for k in names} for _ in range(2))
    silu = lambda h: h * torch.sigmoid(h)  # noqa: E731
    dsilu = lambda h: torch.sigmoid(h) * (1 + h * (1 - torch.sigmoid(h)))  # noqa: E731

    def forward(xb):
        h1 = q(xb) @ q(p["W1"]).T.contiguous() + p["b1"]
        h2 = q(silu(h1)) @ q(p["W2"]).T.contiguous() + p["b2"]
        return h1, h2, q(silu(h2)) @ q(p["W3"]).T.contiguous() + p["b3"]

    losses, g = [], {}
    for step, b0 in enumerate(range(0, x.shape[0], 64), 1):
        xb, tb = x[b0:b0 + 64], t[b0:b0 + 64]
        h1, h2, y = forward(xb)
        losses.append(float(((y - tb) ** 2).mean()))
        dy = 2 * (y - tb) / y.numel()
        d2 = (q(dy) @ q(p["W3"])) * dsilu(h2)
        d1 = (q(d2) @ q(p["W2"])) * dsilu(h1)
        g = {"W3": q(dy).T.contiguous() @ q(silu(h2)), "b3": dy.sum(0),
             "W2": q(d2).T.contiguous() @ q(silu(h1)), "b2": d2.sum(0),
             "W1": q(d1).T.contiguous() @ q(xb), "b1": d1.sum(0)}
        for k in names:
            m[k] = 0.9 * m[k] + 0.1 * g[k]
            v[k] = 0.999 * v[k] + 0.001 * g[k] ** 2
            p[k] = p[k] - 1e-3 * (m[k] / (1 - 0.9 ** step)) / ((v[k] / (1 - 0.999 ** step)).sqrt() + 1e-8)
    host = lambda d: {k: a.cpu().numpy() for k, a in d.items()}  # noqa: E731
    return {"loss": losses, "y": forward(x)[2], "params": host(p), "grads": host(g)}


def exact(case, seed):
    op = case["op"]
    if op == "mlp":
        return _plain_network(case, seed)
    if op == "batch":
        t, xs = _batch_start(case, seed)
        return [_Plain(c).step(t, TAU, case["s"], x) for c, x in zip(_batch_cases(case), xs)]
    if op == "galerkin":
        pl = _Plain(_mesh("c1", case["n"]))
        S, f = _window(pl.free.numel(), case["k"], seed)
        R = torch.stack([pl.mul(s) for s in S])
        c = torch.linalg.solve((S @ R.T.contiguous()).cpu(), (S @ pl.mul(f)).cpu())
        return {"x0": S.T.contiguous() @ c.to(DEV), "kept": None}
    mesh = _mesh(case["recipe"], case["n"], case.get("relabel", False))
    t, x = _start(mesh, seed)
    if op == "rhs":
        return _Plain(mesh, matrix=False).rhs(t, x)
    pl = _Plain(mesh)
    if op == "solve":
        b = pl.rhs(t, x)
        return pl.solve(b, torch.zeros_like(b))
    return pl.step(t, TAU, case["s"], x)
