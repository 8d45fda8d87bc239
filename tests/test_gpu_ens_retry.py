"""An eager ensemble step that one size class fails leaves the classes behind it as if
it had not been called: the same step, taken again once the cause is gone, is the step
of an ensemble that never failed, bit for bit, and the captured pressure system is
still that of the last completed step.

The first class is made to fail by overwriting its fields with NaN (the workspace is
the caller's) and mended by putting the former bytes back.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CAPTURED = ("FIELD_PSOLVE_B", "FIELD_PSOLVE_X", "FIELD_PSOLVE_W", "FIELD_USTAR")


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1404_0959_amd.pisoc as P
    P.lib()
    return P


def values(P, ens, m, bits):
    return {b: ens.get(m, b).cpu().numpy() for b in bits}


@pytest.mark.parametrize("precision,extra", [
    ("fp64", {}), ("fp32", {}), ("fp64", dict(guess="previous")), ("fp32", dict(guess="previous")),
    ("fp64", dict(capture=True)), ("fp32", dict(guess="previous", capture=True)),
])
def test_classes_after_a_failed_one_can_be_retried(P, precision, extra):
    import torch
    from paper_1404_0959_amd.inputs import make_hit_case
    extra = dict(extra)
    guess = extra.pop("guess", None)
    capture = extra.pop("capture", False)
    kw = dict(p_tol=1e-6, p_maxit=60, cfl=0.5, capture=capture)
    if precision == "fp32":
        kw.update(precision=P.FP32_REFINED, inner_tol=1e-3)
    if guess:
        kw.update(guess=P.GUESS_PREVIOUS)
    cs = [make_hit_case(n, 30 + m, mach=0.2, stokes=(0.1,)) for m, n in enumerate((16, 24, 40))]
    good, ens = P.Ensemble(cs, **kw), P.Ensemble(cs, **kw)
    for e in (good, ens):
        st, _ = e.step(2, mode=P.ENS_EAGER)
        assert st in (P.OK, P.WARN_DUST)
    bits = [getattr(P, f) for f in CAPTURED] if capture else []
    before = [values(P, ens, m, bits) for m in range(3)]

    # the first class's region of the workspace, past the device state at its start
    size = P.lib().pisoc_ens_workspace_bytes(ens.prms, 1)
    region = ens.ws[65536:size]
    torch.cuda.synchronize()
    kept = region.clone()
    region.fill_(0xff)
    torch.cuda.synchronize()
    st, _ = ens.step(1, mode=P.ENS_EAGER, raise_on_error=False)
    assert st < 0
    region.copy_(kept)
    torch.cuda.synchronize()
    assert ens.times() == good.times()
    for m in (1, 2):
        for b, v in values(P, ens, m, bits).items():
            assert np.array_equal(v, before[m][b]), (m, b)

    for _ in range(2):
        (sa, ia), (sb, ib) = (e.step(1, mode=P.ENS_EAGER) for e in (good, ens))
        assert sa == sb
        for m in (1, 2):
            assert ia[m] == ib[m], m
    state = [P.FIELD_RHO, P.FIELD_U, P.FIELD_RHO_P]
    for m in (1, 2):
        a, b = values(P, good, m, state + bits), values(P, ens, m, state + bits)
        for k in a:
            assert np.array_equal(a[k], b[k]), (m, k)
