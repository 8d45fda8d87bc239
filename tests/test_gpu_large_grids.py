"""Grids beyond 256 cells a side, at the sizes where the choice of a kernel or its split
changes: rows cut into four segments and more, flattened rows in blocks of more than
512 threads (two w halo cells per thread), the 64-wide tiles, the 16-wide tiles, and
cuts of z into chunks that do not divide n.
"""
import math
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1404_0959_amd.pisoc as P
    P.lib()
    return P


@pytest.mark.parametrize("n", [257, 300, 320, 336, 400, 448])
def test_cg_matches_oracle(P, ora, n):
    """The first iterations of the FP64 solve (one and two x updates per launch, the
    last one at the cap) against the oracle's, to 1e-12 of the solution as for the
    smaller grids: the two differ by the order of the FP64 sums."""
    import torch
    rng = np.random.default_rng(500 + n)
    psidt = 50.0 * (1.0 + 0.2 * rng.random((n, n, n)))
    w = 0.01 * (1.0 + 0.2 * rng.random((n, n, n)))
    b = rng.standard_normal((n, n, n))
    kf = ora.kfaces(w)
    d = [torch.as_tensor(a, device="cuda") for a in (psidt, w, b)]
    for maxit in (2, 3):
        xo, _, rel_o = ora.pcg(psidt, kf, b, tol=1e-14, maxit=maxit)
        xg, it_g, rel_g, st = P.helm_solve(*d, tol=1e-14, maxit=maxit)
        assert st == P.WARN_NOT_CONVERGED and it_g == maxit
        assert abs(rel_g - rel_o) <= 1e-9 * rel_o
        assert np.max(np.abs(xg.cpu().numpy() - xo)) <= 1e-12 * np.max(np.abs(xo))


def flow(n, seed):
    """A few random modes and one dust class, made on the GPU."""
    import torch
    g = np.random.default_rng(seed)
    x = torch.arange(n, device="cuda", dtype=torch.float64) * (2 * math.pi / n)
    X, Y, Z = x[None, None, :], x[None, :, None], x[:, None, None]

    def modes(k):
        return sum(float(g.uniform(0.5, 1.0)) * torch.sin(
            int(g.integers(-4, 5)) * X + int(g.integers(-4, 5)) * Y + int(g.integers(1, 5)) * Z +
            float(g.uniform(0, 6.28))) for _ in range(k))
    rho = 1.0 + 0.01 * modes(3)
    rho_p = 0.1 + 0.02 * modes(3)
    return SimpleNamespace(n=n, rho=rho, u=torch.stack([modes(4) for _ in range(3)]), rho_p=rho_p[None],
                           gamma=1.4, C=4.0, mu=1e-3, tau_p=(0.02,))


@pytest.mark.parametrize("precision,n", [
    ("fp64", 290), ("fp64", 320), ("fp64", 336), ("fp32", 257), ("fp32", 320), ("fp32", 352), ("fp32", 385),
    ("fp32", 528),
])
def test_step_matches_gathered(P, monkeypatch, precision, n):
    """A step against the gathered kernels (PISOC_UNTILED=1), with the bounds of the same
    comparison on smaller grids: 1e-11 of the spread in FP64; in FP32 5e-5 of it plus
    16 FP32 ulps of the magnitude."""
    import torch
    case = flow(n, n)
    kw = dict(p_tol=1e-9) if precision == "fp64" else dict(
        p_tol=1e-6, precision=P.FP32_REFINED, inner_tol=1e-6)
    bits = [P.FIELD_RHO, P.FIELD_U, P.FIELD_PHI, P.FIELD_P, P.FIELD_RHO_P]
    runs = []
    for untiled in (False, True):
        if untiled:
            monkeypatch.setenv("PISOC_UNTILED", "1")
        s = P.Solver.from_case(case, **kw)
        st, info = s.step(1)
        assert st in (P.OK, P.WARN_DUST)
        runs.append(([s.get(b) for b in bits], info[0]))
        s.close()
        del s
    (fa, ia), (fb, ib) = runs
    assert ia["pcg_iters"] == ib["pcg_iters"] and ia["flags"] == ib["flags"]
    assert abs(ia["dt"] / ib["dt"] - 1) <= (1e-12 if precision == "fp64" else 1e-6)
    tol, ulps = (1e-11, 0.0) if precision == "fp64" else (5e-5, 16 * np.finfo(np.float32).eps)
    for bit, a, b in zip(bits, fa, fb):
        spread = float((b - b.mean()).abs().max())
        bound = tol * spread + ulps * float(b.abs().max())
        worst = float((a - b).abs().max())
        assert worst <= bound, (bit, worst, bound)
    del runs, fa, fb
    torch.cuda.empty_cache()


@pytest.mark.parametrize("precision,n", [("fp64", 400), ("fp32", 528)])
def test_multiples_of_16_never_gather(P, precision, n):
    """The CG of a multiple of 16 marches over planes at every size (the gathered form
    reads each stencil again from the caches and reports no planes)."""
    import torch
    one = torch.ones((n, n, n), device="cuda", dtype=torch.float64)
    case = SimpleNamespace(n=n, rho=one, u=torch.zeros((3, n, n, n), device="cuda", dtype=torch.float64),
                           rho_p=None, gamma=1.4, C=1.0, mu=1e-3, tau_p=())
    kw = dict(precision=P.FP32_REFINED, inner_tol=1e-3) if precision == "fp32" else {}
    ens = P.Ensemble([case], dt_fixed=1e-3, p_tol=1e-6, **kw)
    cls = ens.classes()[0]
    assert cls["cg_cells_z"] > 0 and cls["tiled_cells_z"] > 0, cls
    ens.close()
    del ens, case, one
    torch.cuda.empty_cache()
