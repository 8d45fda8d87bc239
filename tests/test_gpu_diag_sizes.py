"""The diagnostics at the sizes where their splits can go wrong: spectra with an odd
and an even number of radix-2 factors and lines that do not divide the tiles of
kx (16, 64, 512); Q and the filtered statistics on columns cut by the grid's edge
in x and y (9, 63, 65, 130), with z chunks that do not divide n.

Bars as in the other diagnostics tests: 1e-12 of the largest shell, of max|Q| and
of each statistic (the sums differ in order only); one cell for the backscatter
count.
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


@pytest.mark.parametrize("n", [16, 64, 512])
def test_spectrum(P, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    u = torch.randn((3, n, n, n), generator=g, device="cuda", dtype=torch.float64)
    E, lam, D = P.spectrum(u)
    k = torch.fft.fftfreq(n, d=1.0 / n, device="cuda", dtype=torch.float64)
    k2 = k[None, None, :] ** 2 + k[None, :, None] ** 2 + k[:, None, None] ** 2
    shell = torch.floor(k2.sqrt() + 0.5).long().reshape(-1)
    want, Dw = torch.zeros(len(E), dtype=torch.float64, device="cuda"), 0.0
    for c in range(3):
        e = (torch.fft.fftn(u[c]) / float(n) ** 3).abs().square() * 0.5
        want += torch.bincount(shell, weights=e.reshape(-1), minlength=len(E))
        Dw += float((k2 * e).sum())
    want = want.cpu().numpy()
    assert np.max(np.abs(E - want)) <= 1e-12 * np.max(want)
    assert abs(D / Dw - 1) <= 1e-12
    assert abs(lam / np.sqrt(5 * want.sum() / Dw) - 1) <= 1e-12


@pytest.mark.parametrize("n", [8, 9, 63, 65, 130])
def test_q_and_filtered_statistics(P, ora, n):
    import torch
    rng = np.random.default_rng(n)
    u = rng.standard_normal((3, n, n, n))
    for _ in range(2):   # smooth it, so that Pi is no sum of noise
        for ax in (1, 2, 3):
            u = 0.25 * (np.roll(u, 1, ax) + np.roll(u, -1, ax)) + 0.5 * u
    d = torch.as_tensor(u, device="cuda")
    q, qmean, divsq = P.qcriterion(d)
    qo = ora.qcriterion(u)
    assert np.max(np.abs(q.cpu().numpy() - qo)) <= 1e-12 * np.max(np.abs(qo))
    assert abs(qmean + 0.5 * divsq) <= 1e-12 * divsq
    got, (want, _, _) = P.sgs_stats(d), ora.sgs_stats(u)
    for a, b in zip(got[:2], want[:2]):
        assert abs(a - b) <= 1e-12 * abs(b)
    # Pi's mean is a sum of both signs: 1e-12 of its terms' size
    assert abs(got[2] - want[2]) <= 1e-12 * max(abs(want[2]), want[1] * np.sqrt(np.mean(qo ** 2) ** 0.5))
    assert abs(got[3] - want[3]) <= 1.0 / n ** 3 + 1e-15
