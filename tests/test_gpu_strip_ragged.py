"""Strips when their height does not divide the row count: the last strip is
completed by uncoupled rows with a zero right-hand side.  Row counts that leave
one, two and three rows over, a single short strip, one strip more than a
wave's 64, both heights, precisions and z conditions; standalone and in solves,
against the per-mode form's bounds.

Tolerances: backward error 1e-14 (FP64) and 2e-6 (FP32) of ||B|| ||z|| + ||r||;
solutions at rtol 1e-10 to 1e-8."""
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


@pytest.mark.parametrize("nr,nz", [(2, 256), (3, 512), (5, 256), (9, 1024), (62, 256), (257, 512), (259, 256),
                                   (1021, 256), (7, 2048)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("rows", [4, 8])
@pytest.mark.parametrize("bc", [0, 0x101])
def test_ragged_strips_backward_error(ax, orc, nr, nz, prec, rows, bc):
    kappa, q = np.full((nr, nz), 1.5), np.full((nr, nz), 0.3)   # constant: A is B
    r = np.random.default_rng(nr + nz).standard_normal((nr, nz))
    oop = orc.operator_from_cells(kappa, q, bc_z=bc & 1, grid=orc.GRID_NODES if bc & 0x100 else orc.GRID_CELLS)
    with ax.op_create(kappa, q, bc_z=bc) as op:
        ax.op_set_strips(op, rows)
        active, count = ax.op_strips_info(op, prec)
        used = 4 if (prec == ax.PREC_FP32 and nz == 2048) else rows
        assert active == (prec == ax.PREC_FP32 or nz <= 1024)
        assert count == (-(-nr // used) if active else 0)
        z = dev(np.zeros((nr, nz)))
        ax.precond_apply(op, dev(r), z, prec=prec)
        z = host(z)
    apply = lambda v: orc.apply(oop, v)  # noqa: E731
    nb = spectral_norm_estimate(apply, (nr, nz), iters=12)
    assert np.linalg.norm(apply(z) - r) / (nb * np.linalg.norm(z) + np.linalg.norm(r)) <= (1e-14 if prec == 0 else 2e-6)


@pytest.mark.parametrize("nr,nz,prec", [(37, 256, 0), (130, 512, 1), (99, 1024, 0), (61, 2048, 1), (519, 256, 1)])
@pytest.mark.parametrize("solver", ["pcg", "pr", "cheb"])
def test_ragged_solves_match_oracle(ax, orc, nr, nz, prec, solver):
    kappa, q = synth.medium_layered(nr, nz, seed=3)
    oop = orc.operator_from_cells(kappa, q)
    b = orc.rhs(oop, synth.ricker_source(nr, nz, 1.0, 1.0, 0.4, 0.05))
    with ax.op_create(kappa, q) as op:
        x = dev(np.zeros((nr, nz)))
        if solver == "cheb":
            st = ax.cheb_solve(op, dev(b), x, rtol=1e-10, prec=prec)
        else:
            st = ax.pcg_solve(op, dev(b), x, rtol=1e-10, prec=prec, flags=ax.FLAG_POLAK_RIBIERE if solver == "pr" else 0)
        assert st["code"] == ax.OK
        assert rel(host(x), orc.solve_reference(oop, b)) <= 1e-8
