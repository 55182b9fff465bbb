"""The element pass over fans of tets (k_kx_fan, k_kx_rate_fan), which large
first-order meshes take, against the FP64 oracle and against the pass over
single tets (EQS_FANS=0, read when a context is created): a mesh whose last
block is nearly empty, shuffled nodes and tets (other rings, other starting
faces), per-block LDS strides, materials with whole exponents (fans) and with
others (their tets one by one). Element by element: an entry is a sum of about
24 terms, each with a relative rounding error of some 20 ulp, so 1e-12 of the
largest entry, the bound the single-tet pass is held to.
"""

import numpy as np
import pytest

import eqsgen
from oracle import fem
from oracle.eqs import EqsOracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1612_09447_amd import EQS_PREC_FP32, Context  # noqa: E402

DEV = torch.device("cuda:0")


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


def relinf(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def make_ctx(case, monkeypatch, fans, generic=False):
    monkeypatch.setenv("EQS_FANS", "1" if fans else "0")
    monkeypatch.setenv("EQS_KX_GENERIC", "1" if generic else "0")
    c = Context(0, torch.cuda.current_stream(DEV))
    c.setup_case(case, precision=EQS_PREC_FP32)
    assert ("fans per block" in c.describe()) == fans
    return c


@pytest.mark.parametrize("n,whole,shuffled,generic", [(59, False, False, False), (59, True, True, False),
                                                      (61, False, False, True)])
def test_fans_match_oracle_and_single_tets(n, whole, shuffled, generic, monkeypatch):
    case = eqsgen.case_c1(n=n, seed=4)
    if whole:
        case.alpha = np.rint(case.alpha)
    if shuffled:
        case.xyz, case.tets, case.dir_nodes, _ = eqsgen.permute_nodes(case.xyz, case.tets, case.dir_nodes, seed=3)
        case.tets, case.tet_mat, _ = eqsgen.shuffle_tets(case.tets, case.tet_mat, seed=5)
    o = EqsOracle(case, dense_limit=0)
    x, t = eqsgen.random_state(case.n_nodes, 6, 2.5), 0.0021
    ref_k = fem.apply_K(case, o.embed(x[o.free], t))
    ref_r = o.stage_rhs(t, x[o.free])
    got = []
    for fans in (True, False):
        with make_ctx(case, monkeypatch, fans, generic) as c:
            y = torch.zeros(case.n_nodes, dtype=torch.float64, device=DEV)
            c.apply_K(t, T(x), y)
            r = torch.zeros(o.n_free, dtype=torch.float64, device=DEV)
            c.stage_rhs(t, T(x[o.free]), r)
            assert relinf(y.cpu().numpy(), ref_k) <= 1e-12
            assert relinf(r.cpu().numpy(), ref_r) <= 1e-12
            # the adaptive controller's stage counts come from the pass's spectral bound
            full = T(0.05 * x)
            st, steps = c.rkc_adaptive(0.0, 4 * case.tau, full, 1e-10, 1e-6, 1e-4, case.tau)
            got.append([q["s"] for q in steps])
    assert got[0] == got[1]


def test_fans_in_a_tuning_record(tmp_path, monkeypatch):
    """The record names fans and replays them; a context that takes none (the
    deterministic pass) takes a block size without timing, the same every time; a
    record of a block size is followed where fans would be taken."""
    case = eqsgen.case_c1(n=59, seed=4)
    rec = tmp_path / "tune.txt"
    monkeypatch.setenv("EQS_TUNE_FILE", str(rec))
    for k in range(2):
        with make_ctx(case, monkeypatch, True) as c:
            assert c.describe().count("fans per block") == 1
            assert ("fans) (tuning record)" in c.describe().replace("a fan)", "a fans)")) == (k == 1)
    line = [ln for ln in rec.read_text().splitlines() if ln.startswith("element ")]
    assert len(line) == 1 and line[0].endswith("\tfans")
    c = Context(0, torch.cuda.current_stream(DEV))
    c.setup_case(case, precision=EQS_PREC_FP32, deterministic=True)
    assert "element: 1024 tets per block (tuning record)" in c.describe()
    c.close()
    rec.write_text(rec.read_text().replace("\tfans", "\t2"))
    with make_ctx(case, monkeypatch, False) as c:
        assert "element: 512 tets per block (tuning record)" in c.describe()
    monkeypatch.setenv("EQS_FANS", "1")
    c = Context(0, torch.cuda.current_stream(DEV))
    c.setup_case(case, precision=EQS_PREC_FP32)
    assert "element: 512 tets per block (tuning record)" in c.describe()
    c.close()
