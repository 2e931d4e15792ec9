"""PCG's iterate after a fixed number of iterations, FP64, against the oracle's:
x is updated one iteration late (in the next SpMV, or in the inverse launch that
finds the solve stopped), so a solve that stops at any iteration has to hold the
full iterate.  Grids at the edges of the SpMV's tiles (256 columns; 2 or 16
rows) and of the transforms' plans, x at an odd 8-byte offset among them.

Tolerance: a few roundings per iteration, amplified by the operators' condition
numbers of at most about 1e6: 1e6 * 16 eps < 1e-8."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel

pytestmark = pytest.mark.gpu
SHAPES = [(3, 2), (5, 16), (33, 64), (17, 128), (36, 256), (35, 512), (18, 1024), (9, 2048), (1030, 256)]


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


def problem(nr, nz):
    kappa, q = synth.medium_layered(nr, nz, seed=nr + nz)
    b = np.random.default_rng(nr * nz).standard_normal((nr, nz))
    return kappa, q, b


@pytest.mark.parametrize("nr,nz", SHAPES)
@pytest.mark.parametrize("maxit", [1, 2, 5])
def test_iterate_matches_oracle(ax, orc, nr, nz, maxit):
    import torch
    kappa, q, b = problem(nr, nz)
    oop = orc.operator_from_cells(kappa, q)
    ref = orc.pcg(oop, b, rtol=1e-12, maxit=maxit)[0]
    with ax.op_create(kappa, q) as op:
        x = torch.zeros(nr * nz + 1, dtype=torch.float64, device="cuda")[1:].view(nr, nz)
        ax.pcg_solve(op, dev(b), x, rtol=1e-12, maxit=maxit, prec=ax.PREC_FP64)
        assert rel(host(x), ref) <= 1e-8


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("flags", [0, 4])
def test_batch_members_that_stop_apart(ax, orc, prec, flags):
    """Members stopping at different iterations (a zero right-hand side, a
    constant medium that converges at once, layered ones)."""
    members = [problem(40, 64), problem(64, 256), problem(30, 512)]
    members[0] = (members[0][0], members[0][1], np.zeros((40, 64)))
    members.append((np.full((24, 128), 2.0), np.full((24, 128), 0.5), members[0][2][:24].repeat(2, axis=1) + 1.0))
    ops = [ax.op_create(k, q) for k, q, _ in members]
    xs = [dev(np.ones(b.shape)) for _, _, b in members]
    ax.batch_solve(ops, [dev(b) for _, _, b in members], xs, rtol=1e-11, prec=prec, flags=flags)
    for (k, q, b), x in zip(members, xs):
        ref = np.zeros(b.shape) if not b.any() else orc.solve_reference(orc.operator_from_cells(k, q), b)
        assert rel(host(x), ref) <= 1e-8 if b.any() else not host(x).any()
    for o in ops:
        o.close()


@pytest.mark.parametrize("maxit", [1, 3])
def test_single_launch_step_holds_the_iterate(ax, orc, maxit):
    """The single-launch form of the iteration ends in the same iterate (FP32
    preconditioner: both forms to its backward error, 2e-6)."""
    kappa, q, b = problem(64, 256)
    with ax.op_create(kappa, q) as op:
        out = []
        for fused in (False, True):
            ax.op_set_fused(op, fused)
            x = dev(np.zeros((64, 256)))
            ax.pcg_solve(op, dev(b), x, rtol=1e-12, maxit=maxit, prec=ax.PREC_FP32)
            out.append(host(x).copy())
        assert ax.op_fused_info(op, ax.FUSED_PCG, want_errors=True)[2] == 0
        assert rel(out[1], out[0]) <= 1e-3
