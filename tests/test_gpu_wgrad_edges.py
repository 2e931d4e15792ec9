"""Weight gradients of the learned guess, tap by tap, on rough fields whose energy lies
where a workgroup's 64-pixel segments meet (columns 63 and 64, 127 and 128, ...) and in
the first and last rows: products of a pixel and its neighbour across two segments, or
across two ranges of rows, are most of what a tap sums.

Tolerance: the library and the oracle round to BF16 at the same places, so they differ
by those roundings that fall the other way; what all roundings together make (the
oracle's rounded gradient against its exact one, layer by layer, at least 2e-2) bounds
that.  It is 0.02 ... 0.3 here, in each layer less than what an oracle
without the products across segments (0.32 ... 1.6) or into the last row (0.23 ... 1.1)
is off by."""
import numpy as np
import pytest

import oracle.nn as onn
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


def taps_of(flat):
    """Per layer the nine taps' weight gradients, [9][cin cout]."""
    return [flat[o:o + 9 * ci * co].reshape(9, -1) for o, ci, co in zip(onn.OFFSETS, onn.CIN, onn.COUT)]


def off(a, ref):
    return (np.linalg.norm(a - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()


@pytest.mark.parametrize("nr,nz", [(4, 64), (2, 128), (3, 128), (65, 128), (20, 1024), (515, 128)])
def test_taps_across_segments_and_rows(ax, orc, nr, nz):
    rng = np.random.default_rng(nr + nz)
    env = np.ones((nr, nz))
    env[:, np.isin(np.arange(nz) % 64, (0, 63))] = 10
    env[[0, -1]] *= 10
    u1, u2, ut, b = (env * rng.standard_normal((nr, nz)) for _ in range(4))
    kappa, q = rng.uniform(1, 4, (nr, nz)), np.full((nr, nz), 0.5)
    params = onn.init_params(5, last_zero=False)
    params[onn.OFFSETS[5]:onn.OFFSETS[5] + 9 * 32] *= 0.001
    oop = orc.operator_from_cells(kappa, q)
    ref, exact = (taps_of(onn.backward(params, onn.forward(params, u1, u2, b, kappa, bf16=r)[1],
                                       lambda e: orc.apply(oop, e), ut)[1]) for r in (True, False))
    with ax.op_create(kappa, q) as op, ax.nn_create(nr, nz, params) as net:
        ax.nn_forward(net, dev(u1), dev(u2), dev(b), dev(kappa), dev(np.zeros((nr, nz))))
        ax.nn_backward(op, net, dev(u1), dev(u2), dev(ut))
        got = taps_of(ax.nn_get_params(net)[1])
    for g, r, e in zip(got, ref, exact):
        assert off(g, r) <= max(2e-2, off(e, r))
