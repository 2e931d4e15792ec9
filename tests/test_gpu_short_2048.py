"""FP32 solves on few rows of 2048 points, which leave the strips: both sides of
the rule (512 rows) and of the row pairing, odd and even counts, both z
conditions and solvers, against the oracle; and a handle whose strips were set,
or whose single launches are on, keeps the strips.

Tolerance: the recurrence residual is reduced to 1e-10 and the operators of
these grids have condition numbers below 1e2 in the preconditioned norm, so the
iterate is good to 1e-8."""
import pytest

import synth
from tests.gpu_util import dev, host, rel

import numpy as np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


@pytest.mark.parametrize("nr", [2, 3, 57, 511, 512, 513])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("solver", ["pcg", "cheb"])
def test_solve_matches_oracle(ax, orc, nr, bc, solver):
    nz = 2048
    kappa, q = synth.medium_layered(nr, nz, seed=nr)
    oop = orc.operator_from_cells(kappa, q, bc_z=bc)
    b = orc.rhs(oop, synth.ricker_source(nr, nz, 1.0, 1.0, 0.4, 0.05))
    ref = orc.solve_reference(oop, b)
    with ax.op_create(kappa, q, bc_z=bc) as op:
        assert ax.op_strips_info(op, ax.PREC_FP32)[0] == (nr > 512)
        for strips in (None, 1):
            if strips is not None:
                ax.op_set_strips(op, strips)
                assert ax.op_strips_info(op, ax.PREC_FP32) == (True, (nr + 3) // 4)
            x = dev(np.zeros((nr, nz)))
            st = (ax.pcg_solve if solver == "pcg" else ax.cheb_solve)(op, dev(b), x, rtol=1e-10, prec=ax.PREC_FP32)
            assert st["code"] == ax.OK
            assert rel(host(x), ref) <= 1e-8


def test_single_launches_keep_the_strips(ax):
    kappa, q = synth.medium_layered(96, 2048, seed=1)
    with ax.op_create(kappa, q) as op:
        ax.op_set_fused(op, True)
        assert ax.op_strips_info(op, ax.PREC_FP32) == (True, 24)
        assert ax.op_fused_info(op, ax.FUSED_PCG)[:2] == (True, 24)
