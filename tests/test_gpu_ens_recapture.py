"""Captured ensemble steps whose graphs are captured again all the time: the two
captured modes in turn on one ensemble, each call dropping the other's graphs right
after they were replayed, with eager steps and reads of the fields in between.  Every
step is bitwise that of an ensemble stepped eagerly throughout.
"""
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


def test_captured_modes_in_turn(P):
    from paper_1404_0959_amd.inputs import make_hit_case
    cs = [make_hit_case(n, 60 + m, mach=0.2, stokes=(0.1,)) for m, n in enumerate((16, 24, 16))]
    a, b = P.Ensemble(cs, p_tol=1e-9), P.Ensemble(cs, p_tol=1e-9)
    for nst, mode in ((3, P.ENS_GRAPH_ONE), (2, P.ENS_GRAPH), (3, P.ENS_GRAPH_ONE), (3, P.ENS_GRAPH_ONE),
                      (1, P.ENS_EAGER), (4, P.ENS_GRAPH), (2, P.ENS_GRAPH_ONE), (2, P.ENS_GRAPH)):
        sa, ia = a.step(nst, mode=P.ENS_EAGER)
        sb, ib = b.step(nst, mode=mode)
        assert sa == sb and sa in (P.OK, P.WARN_DUST)
        for m in range(len(cs)):
            assert ia[m]["pcg_iters"] == ib[m]["pcg_iters"] and ia[m]["t"] == ib[m]["t"], m
            for bit in (P.FIELD_RHO, P.FIELD_U, P.FIELD_RHO_P):
                assert np.array_equal(a.get(m, bit).cpu().numpy(), b.get(m, bit).cpu().numpy()), (m, bit)
    b.close()
    a.close()
