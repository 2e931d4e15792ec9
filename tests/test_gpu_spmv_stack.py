"""PCG on long grids of short rows, whose SpMV workgroups take several tiles one
above the other: both sides of the rule (two tiles from 1024 rows), tiles that do
not divide the row count, stacks limited by the rows and by the workgroup, both
forms of beta, FP64, the iterate after one and four iterations against the
oracle's.

Tolerance: the preconditioner's backward error of 1e-14 times condition numbers of
at most 1e8 (4 nr^2 and a contrast of 10)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


@pytest.mark.parametrize("nr,nz", [(1023, 32), (1024, 32), (1025, 16), (1537, 128), (1539, 64), (2561, 32), (2050, 8),
                                   (3077, 2)])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("polak", [False, True])
def test_iterate_matches_oracle(ax, orc, nr, nz, bc, polak):
    kappa, q = synth.medium_layered(nr, nz, seed=nr)
    b = np.random.default_rng(nr * nz).standard_normal((nr, nz))
    oop = orc.operator_from_cells(kappa, q, bc_z=bc)
    with ax.op_create(kappa, q, bc_z=bc) as op:
        for maxit in (1, 4):
            ref = orc.pcg(oop, b, rtol=1e-12, maxit=maxit)[0]
            x = dev(np.zeros((nr, nz)))
            ax.pcg_solve(op, dev(b), x, rtol=1e-12, maxit=maxit, prec=ax.PREC_FP64,
                         flags=ax.FLAG_POLAK_RIBIERE if polak else 0)
            assert rel(host(x), ref) <= 1e-6
