"""The last round of the Laguerre recurrences, which steps the harmonics that are left up to
a multiple of 16: n on both sides of those multiples, in one round and in a second.

Tolerance: as for the functions themselves, a few roundings per step of the recurrence, at
most 50 n eps of the largest term."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps
COUNTS = [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 64, 66, 79, 80, 81, 112, 113, 127, 128]


@pytest.mark.parametrize("n", COUNTS)
def test_projection(ax, orc, n):
    nt, eta, tmax = 129, 300.0, 0.4
    t = np.linspace(0.0, tmax, nt)
    f = np.random.default_rng(n).standard_normal(nt)
    w = np.full(nt, tmax / (nt - 1))
    w[0] = w[-1] = 0.5 * w[0]
    for alpha in (0, 5):
        psi = orc.laguerre_psi(n, alpha, eta, t)
        tol = 50 * (n + nt) * EPS * np.abs(psi).max() * np.abs(w * f).sum()
        got = ax.laguerre_coeffs_alpha(n, alpha, eta, f, tmax)
        assert np.abs(got - psi @ (w * f)).max() <= tol
        np.testing.assert_array_equal(ax.laguerre_coeffs_alpha_noalloc(n, alpha, eta, f, tmax), got)


@pytest.mark.parametrize("n", COUNTS)
def test_synthesis(ax, orc, n):
    import torch
    nrec, nt, alpha, eta, tmax = 5, 130, 5, 300.0, 0.4
    Q = np.random.default_rng(n).standard_normal((n, nrec))
    phi = orc.laguerre_synthesis(n, alpha, eta, np.linspace(0.0, tmax, nt))
    out = torch.empty((nrec, nt), dtype=torch.float64, device="cuda")
    ax.laguerre_synth(alpha, eta, dev(Q), nt, tmax, out)
    assert np.abs(host(out) - Q.T @ phi).max() <= 50 * n * EPS * (np.abs(Q).T @ np.abs(phi)).max()
