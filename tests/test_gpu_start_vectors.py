"""Edges of the start-vector kernels: batches around the network's chunk of 64
samples, windows of one to sixteen columns over row counts that are no multiple
of a wavefront's. Oracles and error scales as in test_gpu_learned."""

import numpy as np
import pytest

import eqsgen
from oracle import mlp as omlp
from oracle.eqs import EqsOracle
from oracle.guess import galerkin_start, pod_from_gram

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1612_09447_amd import EQS_PREC_FP64, Context, Mlp  # noqa: E402
from test_gpu_learned import TOL, abs_forward, elementwise, grad_scales, params64  # noqa: E402

DEV = torch.device("cuda:0")


def F32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device=DEV)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B", [1, 15, 63, 65, 129, 200])
def test_network_batches_around_a_chunk(B, bf16):
    p = eqsgen.mlp_init(7)
    net = Mlp(p, bf16=bf16, lr=1e-3, stream=torch.cuda.current_stream(DEV))
    rng = np.random.default_rng(B)
    x = rng.normal(size=(B, 32)).astype(np.float32)
    t = rng.normal(size=(B, 16)).astype(np.float32)
    y = torch.full((B + 1, 16), 7.0, dtype=torch.float32, device=DEV)
    net.forward(F32(x), y[:B])
    ref, scale = abs_forward(params64(p), x.astype(np.float64), bf16)
    elementwise(y[:B].cpu().numpy(), ref, scale, TOL[bf16], f"forward B={B} bf16={bf16}")
    assert bool((y[B] == 7.0).all())  # nothing past the batch
    net.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B", [1, 2, 15, 31, 32])
def test_network_trains_alike_on_a_batch_and_on_two_copies_of_it(B, bf16):
    """The mean loss and its gradients are those of the batch. Every sample's terms
    are the same numbers, times an exact power of two, so only the order of the
    sums differs: at most 64 terms, 2^-24 of their magnitudes each, so within 4e-6
    of the sum of magnitudes; against the oracle's magnitudes, which know the output
    errors y - t to FP32 only, twice that."""
    rng = np.random.default_rng(40 + B)
    x = rng.normal(size=(B, 32)).astype(np.float32)
    t = rng.normal(size=(B, 16)).astype(np.float32)
    out = []
    for copies in (1, 2):
        net = Mlp(eqsgen.mlp_init(7), bf16=bf16, lr=1e-3, stream=torch.cuda.current_stream(DEV))
        loss = net.train_step(F32(np.tile(x, (copies, 1))), F32(np.tile(t, (copies, 1))))
        out.append((loss, net.get()[1]))
        net.close()
    assert abs(out[0][0] - out[1][0]) <= 1e-6 * out[0][0]
    sc = grad_scales(params64(eqsgen.mlp_init(7)), x.astype(np.float64), t.astype(np.float64), bf16)
    for k in omlp.NAMES:
        elementwise(out[0][1][k], np.asarray(out[1][1][k], np.float64), sc[k], 8e-6, f"gradient {k} B={B} bf16={bf16}")


@pytest.mark.parametrize("n", [6, 9, 13])
@pytest.mark.parametrize("k", [1, 2, 7, 15, 16])
def test_window_of_k_columns(n, k):
    """Random windows are well conditioned (sigma_1 / sigma_k below 10), so the basis
    and the reduced solve lose two digits of FP64 at most: 1e-10 as for the windows
    of test_gpu_learned."""
    case = eqsgen.case_c1(n=n, seed=1)
    o = EqsOracle(case)
    rng = np.random.default_rng(100 * n + k)
    S = rng.standard_normal((o.n_free, k))
    r = rng.standard_normal(o.n_free)
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)  # noqa: E731
    with Context(0, torch.cuda.current_stream(DEV)) as c:
        c.setup_case(case, precision=EQS_PREC_FP64)
        x0 = torch.full((o.n_free,), float("nan"), dtype=torch.float64, device=DEV)
        m = c.galerkin_start(T(S.T), T((o.M_II @ S).T), T(r), x0)
    V, _, _ = pod_from_gram(S, 16)
    want = galerkin_start(V, o.M_II, r)
    assert m == V.shape[1] == k
    assert np.linalg.norm(x0.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
