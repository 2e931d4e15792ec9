"""The projection onto and the synthesis from the Laguerre functions at the
edges of their work split: rounds of 64 harmonics, groups of 64 samples,
receivers per wave, and more sample groups than partial sums.

Tolerance: a three-term recurrence step adds a few roundings, and n of them
add up at most linearly in the oscillatory region, so both sides stay within
50 n eps of the largest term."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


@pytest.mark.parametrize("n,nt,alpha,eta", [(1, 3, 0, 10.0), (63, 64, 5, 300.0), (64, 65, 1, 300.0),
                                            (65, 127, 0, 60.0), (129, 129, 3, 300.0), (2000, 1000, 5, 300.0),
                                            (100000, 385, 2, 5.0)])
def test_projection_matches_oracle_functions(ax, orc, n, nt, alpha, eta):
    tmax = 0.4
    t = np.linspace(0.0, tmax, nt)
    f = np.random.default_rng(n + nt).standard_normal(nt)
    w = np.full(nt, tmax / (nt - 1))
    w[0] = w[-1] = 0.5 * w[0]
    psi = orc.laguerre_psi(n, alpha, eta, t)
    ref = psi @ (w * f)
    tol = 50 * (n + nt) * EPS * np.abs(psi).max() * np.abs(w * f).sum()
    got = ax.laguerre_coeffs_alpha(n, alpha, eta, f, tmax)
    assert np.abs(got - ref).max() <= tol
    if n + nt <= 131072:
        np.testing.assert_array_equal(ax.laguerre_coeffs_alpha_noalloc(n, alpha, eta, f, tmax), got)
    if alpha == 0:
        assert np.abs(ax.laguerre_coeffs(n, eta, f, tmax) - ref).max() <= tol


@pytest.mark.parametrize("n,nrec,nt,alpha", [(1, 1, 2, 0), (64, 3, 64, 5), (65, 33, 65, 1), (200, 70, 1300, 5),
                                             (129, 260, 2001, 0)])
def test_synthesis_matches_oracle_functions(ax, orc, n, nrec, nt, alpha):
    import torch
    eta, tmax = 300.0, 0.4
    t = np.linspace(0.0, tmax, nt)
    Q = np.random.default_rng(n + nrec).standard_normal((n, nrec))
    phi = orc.laguerre_synthesis(n, alpha, eta, t)
    ref = Q.T @ phi
    out = torch.empty((nrec, nt), dtype=torch.float64, device="cuda")
    ax.laguerre_synth(alpha, eta, dev(Q), nt, tmax, out)
    assert np.abs(host(out) - ref).max() <= 50 * n * EPS * (np.abs(Q).T @ np.abs(phi)).max()
