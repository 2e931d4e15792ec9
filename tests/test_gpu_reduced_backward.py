"""The reduced systems with factored coefficients by their backward error, where their
lanes' rows change form: one strip, fewer strips than lanes, 64 lanes of 1, 2, 4, 8 and
16 rows, exactly and one more.

Tolerance: ||B z - r|| / (||B|| ||z|| + ||r||) of 1e-14 (FP64) and 2e-6 (FP32), the
preconditioner's bounds at any size."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, spectral_norm_estimate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strips", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("prec", [0, 1])
def test_backward_error(ax, orc, strips, prec):
    nr, nz = 4 * strips, 256
    kappa, q = np.full((nr, nz), 1.5), np.full((nr, nz), 0.3)   # constant: A is B
    r = np.random.default_rng(strips).standard_normal((nr, nz))
    oop = orc.operator_from_cells(kappa, q)
    with ax.op_create(kappa, q) as op:
        assert ax.op_strips_info(op, prec) == (True, strips)
        z = dev(np.zeros((nr, nz)))
        ax.precond_apply(op, dev(r), z, prec=prec)
        z = host(z)
    apply = lambda v: orc.apply(oop, v)  # noqa: E731
    nb = spectral_norm_estimate(apply, (nr, nz), iters=12)
    assert np.linalg.norm(apply(z) - r) / (nb * np.linalg.norm(z) + np.linalg.norm(r)) <= (1e-14 if prec == 0 else 2e-6)
