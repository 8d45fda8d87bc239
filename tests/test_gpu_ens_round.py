"""An eager ensemble step tries its size classes at the same time and commits them
in their order: the step a class fails, the classes before it have advanced and
those after it keep their state, whatever order they ended in.
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


@pytest.mark.parametrize("sizes,bad", [((32, 16, 24), 1), ((16, 48), 0), ((20, 32, 16, 24, 40, 36), 3)])
def test_classes_after_a_failed_one_keep_their_state(P, sizes, bad):
    from paper_1404_0959_amd.inputs import make_hit_case
    cs = [make_hit_case(n, 70 + m, mach=0.2, stokes=(0.1,)) for m, n in enumerate(sizes)]
    kw = dict(p_tol=1e-7, p_maxit=60, cfl=0.5)
    good = P.Ensemble(cs, **kw)
    st, _ = good.step(1, mode=P.ENS_EAGER)
    assert st in (P.OK, P.WARN_DUST)
    cs[bad].u[0, 1, 2, 3] = np.nan
    ens = P.Ensemble(cs, **kw)
    before = [ens.fields(m, P.FIELD_U)[P.FIELD_U].cpu().numpy() for m in range(len(sizes))]
    st, _ = ens.step(1, mode=P.ENS_EAGER, raise_on_error=False)
    assert st < 0 and ens.last_error()
    t, tg = ens.times(), good.times()
    for m in range(len(sizes)):
        u = ens.fields(m, P.FIELD_U)[P.FIELD_U].cpu().numpy()
        if m < bad:   # the step of the ensemble without the fault, bit for bit
            assert t[m] == tg[m] > 0.0
            assert np.array_equal(u, good.fields(m, P.FIELD_U)[P.FIELD_U].cpu().numpy())
        else:
            assert t[m] == 0.0
            assert np.array_equal(u, before[m], equal_nan=True)
