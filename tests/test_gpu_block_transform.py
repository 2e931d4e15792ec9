"""Long rows whose transforms run block-wide (2048 points in FP64, 4096 in
both precisions): odd and even row counts on both sides of the pairing rule
(512 rows), both z conditions, standalone and in a solve.

Tolerances: the FP64 preconditioner is backward stable to 1e-14 of
||B|| ||z|| + ||r||, the FP32 one to 2e-6 (a few eps32 log2 N per transform and
elimination); iterates as in the fixed-iteration test."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel, spectral_norm_estimate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


@pytest.mark.parametrize("prec,nr,nz", [(0, 3, 2048), (0, 510, 2048), (0, 513, 2048), (0, 4, 4096), (0, 514, 4096),
                                        (1, 5, 4096), (1, 511, 4096), (1, 515, 4096)])
@pytest.mark.parametrize("bc", [0, 1])
def test_preconditioner_backward_error(ax, orc, prec, nr, nz, bc):
    kappa, q = np.full((nr, nz), 1.5), np.full((nr, nz), 0.3)   # constant: A is B
    r = np.random.default_rng(nr + nz).standard_normal((nr, nz))
    oop = orc.operator_from_cells(kappa, q, bc_z=bc)
    with ax.op_create(kappa, q, bc_z=bc) as op:
        z = dev(np.zeros((nr, nz)))
        ax.precond_apply(op, dev(r), z, prec=prec)
        z = host(z)
    apply = lambda v: orc.apply(oop, v)  # noqa: E731
    nb = spectral_norm_estimate(apply, (nr, nz), iters=12)
    err = np.linalg.norm(apply(z) - r) / (nb * np.linalg.norm(z) + np.linalg.norm(r))
    assert err <= (1e-14 if prec == 0 else 2e-6)


@pytest.mark.parametrize("prec,nr,nz", [(0, 7, 2048), (0, 513, 2048), (1, 6, 4096), (1, 513, 4096)])
@pytest.mark.parametrize("solver", ["pcg", "cheb"])
def test_solve_matches_oracle(ax, orc, prec, nr, nz, solver):
    kappa, q = synth.medium_layered(nr, nz, seed=5)
    b = orc.rhs(orc.operator_from_cells(kappa, q), synth.ricker_source(nr, nz, 1.0, 1.0, 0.4, 0.05))
    ref = orc.solve_reference(orc.operator_from_cells(kappa, q), b)
    with ax.op_create(kappa, q) as op:
        x = dev(np.zeros((nr, nz)))
        st = (ax.pcg_solve if solver == "pcg" else ax.cheb_solve)(op, dev(b), x, rtol=1e-10, prec=prec)
        assert st["code"] == ax.OK
        assert rel(host(x), ref) <= 1e-8
