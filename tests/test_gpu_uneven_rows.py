"""FP32 preconditioners on right-hand sides whose rows differ by a factor of 1e5 from one
to the next, on a grid so coarse in r (l_r = 1e6) that rows hardly couple: each row of the
result is as accurate by its own size as a large one, where rows are transformed one by
one.  (Two rows through one complex FFT would leave 6e-8 of the larger one in the
smaller, 6e-3 of it and more.)

Tolerance: two transforms and a solve of some 2 eps32 log2(N) each, 3 x 2 x 12 x 6e-8
< 1e-5 of the row's norm."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


def problem(orc, nr, nz, bc, first):
    kappa, q = np.full((nr, nz), 1.5), np.full((nr, nz), 1.0)
    r = np.random.default_rng(nr + nz).standard_normal((nr, nz))
    r[first::2] *= 1e-5
    return kappa, q, r, orc.operator_from_cells(kappa, q, lr=1e6, bc_z=bc)


def worst_row(z, ref):
    return (np.linalg.norm(z - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()


@pytest.mark.parametrize("nr,nz", [(512, 2048), (515, 2048), (700, 2048), (513, 4096)])
@pytest.mark.parametrize("bc", [0, 1])
def test_apply(ax, orc, nr, nz, bc):
    kappa, q, r, oop = problem(orc, nr, nz, bc, nr % 2)
    with ax.op_create(kappa, q, lr=1e6, bc_z=bc) as op:
        ax.op_set_strips(op, 0)
        z = dev(np.zeros((nr, nz)))
        ax.precond_apply(op, dev(r), z, prec=ax.PREC_FP32)
        assert worst_row(host(z), orc.precond(oop, r)) <= 1e-5


# one step of PCG from zero is the preconditioned residual times a scalar: block-wide
# rows, and grids whose solve is one workgroup
@pytest.mark.parametrize("nr,nz", [(512, 2048), (256, 16), (127, 32), (64, 64), (63, 64), (31, 128), (2, 128)])
@pytest.mark.parametrize("bc", [0, 1])
def test_first_iterate(ax, orc, nr, nz, bc):
    kappa, q, r, oop = problem(orc, nr, nz, bc, nr % 2)
    with ax.op_create(kappa, q, lr=1e6, bc_z=bc) as op:
        x = dev(np.zeros((nr, nz)))
        ax.pcg_solve(op, dev(r), x, rtol=1e-14, maxit=1, prec=ax.PREC_FP32)
        assert worst_row(host(x), orc.pcg(oop, r, rtol=1e-14, maxit=1)[0]) <= 1e-5
