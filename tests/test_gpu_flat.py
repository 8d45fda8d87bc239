"""The kernels that work on flattened full x-rows, at the grid sizes where their
split can go wrong: rows shorter than a wavefront, a last block of a plane with
fewer rows than the others (17, 33, 47, 65, 131), one row fewer than a block
holds, chunks of z that do not divide n, both halo splits (one and two w cells
per thread) and the largest row counts per block.
"""
import math

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


@pytest.mark.parametrize("n", [9, 16, 17, 33, 47, 64, 65, 100, 131, 192])
def test_cg_matches_oracle(P, ora, n):
    """Iteration for iteration: the same count, residual and solution as the FP64
    oracle's Jacobi-PCG.  The two differ by the order of the FP64 sums only: 1e-12
    of the solution, as for the other forms."""
    import torch
    rng = np.random.default_rng(300 + n)
    psidt = 50.0 * (1.0 + 0.2 * rng.random((n, n, n)))
    w = 0.01 * (1.0 + 0.2 * rng.random((n, n, n)))
    b = rng.standard_normal((n, n, n))
    xo, it_o, rel_o = ora.pcg(psidt, ora.kfaces(w), b, tol=1e-10, maxit=500)
    d = lambda a: torch.as_tensor(a, device="cuda")
    xg, it_g, rel_g, st = P.helm_solve(d(psidt), d(w), d(b), tol=1e-10, maxit=500)
    assert st == P.OK and it_g == it_o, (it_g, it_o)
    assert abs(rel_g - rel_o) <= 1e-3 * rel_o
    assert np.max(np.abs(xg.cpu().numpy() - xo)) <= 1e-12 * np.max(np.abs(xo))
    # from a start other than zero, stopped by the cap (odd and even x updates)
    x0 = rng.standard_normal((n, n, n))
    for maxit in (2, 3):
        xo, _, _ = ora.pcg(psidt, ora.kfaces(w), b, x0=x0, tol=1e-14, maxit=maxit)
        xg, it_g, _, st = P.helm_solve(d(psidt), d(w), d(b), x0=d(x0), tol=1e-14, maxit=maxit)
        assert st == P.WARN_NOT_CONVERGED and it_g == maxit
        assert np.max(np.abs(xg.cpu().numpy() - xo)) <= 1e-12 * np.max(np.abs(xo))


def _fields(P, s, classes):
    bits = P.FIELD_RHO | P.FIELD_U | P.FIELD_PHI | P.FIELD_P | (P.FIELD_RHO_P if classes else 0)
    return {k: v.cpu().numpy() for k, v in s.fields(bits).items()}


@pytest.mark.parametrize("precision,n,variant", [
    ("fp64", 65, {}), ("fp64", 70, {}), ("fp64", 128 - 1, {}),
    ("fp64", 70, dict(two_way=True, gravity=(0.1, 0.0, -1.0))),
    ("fp64", 75, dict(bdf2=True)), ("fp64", 75, dict(mom_tol=1e-8)), ("fp64", 70, dict(fourier=True)),
    ("fp32", 66, {}), ("fp32", 101, {}), ("fp32", 200, {}),
    ("fp32", 70, dict(two_way=True, gravity=(0.1, 0.0, -1.0))),
])
def test_step_matches_gathered(P, monkeypatch, precision, n, variant):
    """Two steps on the flat-row kernels against the gathered ones
    (PISOC_UNTILED=1): both call the same cell arithmetic, so the CG iteration
    counts and flags agree and the fields agree to rounding, with the bounds of the
    tiled kernels' comparison (FP64: 1e-11 of the spread; FP32: 5e-5 of the spread
    plus 16 FP32 ulps of the magnitude)."""
    from paper_1404_0959_amd.inputs import make_hit_case
    variant = dict(variant)
    classes = 0 if variant.get("fourier") else 2
    case = make_hit_case(n, 7, mach=0.5, stokes=(0.1, 0.4)[:classes])
    if variant.pop("fourier", False):
        variant["fourier"] = dict(R=1.0, cv=2.5, kappa=1e-3, T0=case.C)
    kw = dict(p_tol=1e-9) if precision == "fp64" else dict(
        p_tol=1e-6, precision=P.FP32_REFINED, inner_tol=1e-6)
    runs = []
    for untiled in (False, True):
        if untiled:
            monkeypatch.setenv("PISOC_UNTILED", "1")
        s = P.Solver.from_case(case, **kw, **variant)
        st, info = s.step(2)
        assert st in (P.OK, P.WARN_DUST)
        runs.append((_fields(P, s, classes), [(i["pcg_iters"], i["flags"], i["mom_iters"]) for i in info],
                     [i["dt"] for i in info]))
        monkeypatch.delenv("PISOC_UNTILED", raising=False)
    (fa, ia, da), (fb, ib, db) = runs
    assert ia == ib
    np.testing.assert_allclose(da, db, rtol=1e-12 if precision == "fp64" else 1e-6)
    tol, ulps = (1e-11, 0.0) if precision == "fp64" else (5e-5, 16 * np.finfo(np.float32).eps)
    for k in fa:
        spread = np.max(np.abs(fb[k] - fb[k].mean()))
        bound = tol * spread + ulps * np.max(np.abs(fb[k]))
        d = np.max(np.abs(fa[k] - fb[k]))
        assert d <= bound, (k, d, bound)


@pytest.mark.parametrize("n", [65, 70, 100])
def test_chebyshev_matches_oracle(P, ora, n):
    """The polynomial-preconditioned solve on flattened rows: the oracle's iteration
    count, residual and solution, as for the other forms."""
    import torch
    rng = np.random.default_rng(400 + n)
    h = 2 * math.pi / n
    w = 0.01 * (1.0 + 0.2 * rng.random((n, n, n)))
    psidt = 3.0 * 0.01 / h ** 2 * (1.0 + 0.2 * rng.random((n, n, n)))
    b = rng.standard_normal((n, n, n))
    xo, it_o, rel_o = ora.pcg_cheb(psidt, ora.kfaces(w), b, tol=1e-10, maxit=500)
    d = lambda a: torch.as_tensor(a, device="cuda")
    xg, it_g, rel_g, st = P.helm_solve(d(psidt), d(w), d(b), tol=1e-10, maxit=500,
                                       precond=P.PRECOND_CHEB)
    assert st == P.OK and it_g == it_o, (it_g, it_o)
    assert abs(rel_g - rel_o) <= 1e-3 * rel_o
    assert np.max(np.abs(xg.cpu().numpy() - xo)) <= 1e-12 * np.max(np.abs(xo))


@pytest.mark.parametrize("precision,n,members", [
    ("fp64", 20, 16), ("fp64", 33, 6), ("fp32", 66, 8), ("fp64", 66, 9),
])
def test_batched_cg_sums_as_a_single_run(P, precision, n, members):
    """A batch's CG blocks march over several of the single grid's z-chunks (with a
    short last march at 33 and 66) and total each chunk by itself: a member's
    solves and fields are bitwise those of a run of its own."""
    from paper_1404_0959_amd.inputs import make_hit_case
    cs = [make_hit_case(n, 50 + m, mach=0.2 if m % 2 else 0.5, stokes=(0.1,)) for m in range(members)]
    kw = dict(precision=P.FP32_REFINED if precision == "fp32" else P.FP64, p_tol=1e-7,
              inner_tol=1e-5, cfl=0.5)
    ens = P.Ensemble(cs, **kw)
    st, infos = ens.step(2, mode=P.ENS_EAGER)
    assert st in (P.OK, P.WARN_DUST)
    for m in (0, members - 1):
        s = P.Solver.from_case(cs[m], **kw)
        st, rec = s.step(2)
        assert st in (P.OK, P.WARN_DUST)
        assert infos[m]["pcg_iters"] == rec[-1]["pcg_iters"]
        a = {k: v.cpu().numpy() for k, v in ens.fields(m, P.FIELD_U | P.FIELD_P).items()}
        b = {k: v.cpu().numpy() for k, v in s.fields(P.FIELD_U | P.FIELD_P).items()}
        for k in a:
            assert np.array_equal(a[k], b[k]), (m, k)
        s.close()
    ens.close()


@pytest.mark.parametrize("precision,n,variant", [
    ("fp64", 129, {}), ("fp64", 193, {}), ("fp64", 200, {}), ("fp32", 130, {}), ("fp32", 193, {}),
    ("fp64", 136, dict(two_way=True, gravity=(0.1, 0.0, -1.0))), ("fp64", 131, dict(bdf2=True)),
    ("fp64", 130, dict(mom_tol=1e-8)), ("fp64", 150, dict(fourier=True)),
])
def test_segmented_step_matches_gathered(P, monkeypatch, precision, n, variant):
    """The same comparison beyond 128, where a block owns segments of its rows: a
    last segment narrower than the others (57 of 72 columns at 129, 49 at 193, 56
    at 200), a last block with fewer rows, and the x halo across the period."""
    test_step_matches_gathered(P, monkeypatch, precision, n, variant)


@pytest.mark.parametrize("n", [130, 161])
def test_segmented_chebyshev_matches_oracle(P, ora, n):
    """As above, with the polynomial's two launches on segments."""
    test_chebyshev_matches_oracle(P, ora, n)


@pytest.mark.parametrize("precision,n,variant", [
    ("fp64", 9, {}), ("fp64", 17, {}), ("fp64", 39, {}), ("fp32", 16, {}), ("fp32", 33, {}),
    ("fp64", 20, dict(two_way=True, gravity=(0.1, 0.0, -1.0))), ("fp64", 24, dict(bdf2=True)),
    ("fp64", 32, dict(fourier=True)),
])
def test_small_fused_passes_match_separate(P, monkeypatch, precision, n, variant):
    """The same comparison below 40: the corrector's and the dust's fused passes on
    the gathered launch against the separate kernels."""
    test_step_matches_gathered(P, monkeypatch, precision, n, variant)
