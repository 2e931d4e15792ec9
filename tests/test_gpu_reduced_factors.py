"""The reduced systems with factored coefficients (strips of four rows) where
their lanes' rows change form: one strip, fewer strips than lanes, 64 lanes of
1, 2, 4, 8 and 16 rows, exactly and one more, in both precisions, against the
per-mode r-solve of the same handle.

Tolerance: two backward-stable solves of the same system differ by the
condition number of its r-lines (about nr^2) times a few eps."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


@pytest.mark.parametrize("strips", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("prec", [0, 1])
def test_factored_reduced_systems(ax, strips, prec):
    nr, nz = 4 * strips, 256
    rng = np.random.default_rng(strips)
    kappa = 1.0 + rng.random((nr, nz))
    r = rng.standard_normal((nr, nz))
    out = []
    with ax.op_create(kappa, np.full((nr, nz), 0.4)) as op:
        for rows in (4, 0):
            ax.op_set_strips(op, rows)
            assert ax.op_strips_info(op, prec) == ((True, strips) if rows else (False, 0))
            z = dev(np.zeros((nr, nz)))
            ax.precond_apply(op, dev(r), z, prec=prec)
            out.append(host(z).copy())
    eps = 2.2e-16 if prec == 0 else 6e-8
    assert rel(out[0], out[1]) <= max(64, nr * nr) * 4 * eps
