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
