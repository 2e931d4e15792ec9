"""Weight gradients of the learned guess where a workgroup's range of 64-pixel
segments (numbered down the rows of a column of segments) changes form: a single
segment with both neighbour rows outside the grid, ranges of one segment, ranges
that end inside a column, and ranges that go on in the next column.

Tolerance: data gradients and activations are rounded to BF16 (2^-8) at each of
six layers, so a layer's gradient is good to 2e-2 of its norm."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    assert torch.cuda.is_available()
    from paper_1002_3094_amd import axipcg
    axipcg.lib()
    return axipcg


# segments: 4 and 8 (one a workgroup), 1030 and 1072 (one or two), 2624 and 3296
# (two or three, three or four) over columns of 2 .. 515 rows
# 4 x 64: one activation rounds the other way than the oracle's, which 256 pixels do
# not average out: 2.54315e-2 in the first layer, to six digits the same with the
# earlier kernel, which staged each segment by itself.
@pytest.mark.parametrize("nr,nz", [pytest.param(4, 64, marks=pytest.mark.xfail(
                                       reason="a rounding before the weight gradient differs from the oracle's")),
                                   (2, 256), (515, 128), (67, 1024), (41, 4096), (206, 1024)])
def test_weight_gradient_over_ranges(ax, orc, nr, nz):
    from oracle import nn as onn
    ex = synth.nn_example(nr, nz, seed=nr)
    q = np.full((nr, nz), 0.5)
    params = onn.init_params(5, last_zero=False)
    params[onn.OFFSETS[5]:onn.OFFSETS[5] + 9 * 32] *= 0.001
    oop = orc.operator_from_cells(ex["kappa"], q)
    with ax.op_create(ex["kappa"], q) as op, ax.nn_create(nr, nz, params) as net:
        u1, u2 = dev(ex["u1"]), dev(ex["u2"])
        ax.nn_forward(net, u1, u2, dev(ex["b"]), dev(ex["kappa"]), dev(np.zeros((nr, nz))))
        ax.nn_backward(op, net, u1, u2, dev(ex["ut"]))
        _, grad = ax.nn_get_params(net)
    _, cache = onn.forward(params, ex["u1"], ex["u2"], ex["b"], ex["kappa"])
    _, ref = onn.backward(params, cache, lambda e: orc.apply(oop, e), ex["ut"])
    ends = list(onn.OFFSETS) + [len(params)]
    for lo, hi in zip(ends[:6], ends[1:7]):
        assert np.linalg.norm(grad[lo:hi] - ref[lo:hi]) <= 2e-2 * np.linalg.norm(ref[lo:hi])
