"""PCG on long grids of short rows with the FP32 preconditioner, whose stacked SpMV reads
z as floats: both forms of beta, stacks that end past the last row, the iterate after one
and four steps, on well-conditioned operators (unit steps, eigenvalues of 1 ... 50 in
the mass-weighted norm) and right-hand sides with most of their energy in the last rows.

Tolerances: x and the recurrence residual take the same p and A p, so b - A x and the
recurrence residual differ by FP64 rounding alone, 1e-12 of ||b||; the iterates differ
from those of an exact preconditioner by its 2e-6 times the condition number (50) for
each step, 4e-4, while a row left out of a stack is off by 3e-2 and more."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nz", [(1024, 32), (1025, 16), (1537, 128), (1539, 64), (2561, 32), (2050, 8), (3077, 2)])
@pytest.mark.parametrize("polak", [False, True])
def test_iterate(ax, orc, nr, nz, polak):
    rng = np.random.default_rng(nr * nz)
    kappa, q = rng.uniform(1.0, 2.0, (nr, nz)), rng.uniform(1.0, 2.0, (nr, nz))
    b = rng.standard_normal((nr, nz))
    b[-7:] *= 30
    oop = orc.operator_from_cells(kappa, q, lr=nr, lz=nz)
    with ax.op_create(kappa, q, lr=nr, lz=nz) as op:
        for maxit in (1, 4):
            x = dev(np.zeros((nr, nz)))
            st = ax.pcg_solve(op, dev(b), x, rtol=1e-12, maxit=maxit, prec=ax.PREC_FP32,
                              flags=(ax.FLAG_POLAK_RIBIERE if polak else 0) | ax.FLAG_TRUE_RESIDUAL)
            assert st["iters"] == maxit and abs(st["relres_true"] - st["relres_rec"]) <= 1e-12
            assert rel(host(x), orc.pcg(oop, b, rtol=1e-12, maxit=maxit)[0]) <= 4e-4
