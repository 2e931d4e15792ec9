"""Kernels that a rule of dispatch replaced are not built any more: the reduced systems
of 4-row strips with recomputed coefficients, more rows a lane than 512 strips of eight
rows need or fewer modes a workgroup than fit, and the Stockham transforms' forms for
rows too long to keep twiddles in LDS.  And the single launch asks for the LDS it uses."""
import re

from tests import _hostcode

DRIVER = r"""
#include <cstdio>
#include "_fake_hip.h"
int main()
{
    for (const std::string &k : fake::kernels()) std::printf("%s\n", k.c_str());
    return 0;
}
"""


def test_replaced_kernels_are_gone(tmp_path_factory):
    names = [re.sub(r"^void axipcg::\(anonymous namespace\)::", "", n)
             for n in _hostcode.run(tmp_path_factory, DRIVER, library=True).split("\n")]
    reduced = [n for n in names if n.startswith("k_strip_reduced<")]
    assert reduced and all(re.match(r"k_strip_reduced<(float, 8, [1248], 8|double, 8, [1248], 4)>\(", n) for n in reduced)
    assert sum(n.startswith("k_zfwd<") for n in names) == 2 * 2 * 3   # z condition, fused or not, FP32 and FP64 in one or two rows


LDS = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    for (int nz : {256, 2048}) {
        const int nr = 512;
        const size_t n = (size_t)nr * nz;
        std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
        axipcg_op_t op = nullptr;
        if (axipcg_op_create(nr, nz, 1, 1, 0, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
        axipcg_op_set_fused(op, 1);
        if (axipcg_precond_apply(op, b.data(), x.data(), AXIPCG_PREC_FP32, nullptr)) return 3;
        if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 1, AXIPCG_PREC_FP32, 0, nullptr, nullptr) < 0) return 4;
        for (const fake::Launch &l : fake::launches)
            if (fake::has(l.kernel, "k_strip_one")) std::printf("%u %zu\n", l.grid.x, l.lds);
        fake::launches.clear();
        axipcg_op_destroy(op);
    }
    return 0;
}
"""


def test_single_launch_lds(tmp_path_factory):
    out = [tuple(map(int, line.split())) for line in _hostcode.run(tmp_path_factory, LDS, library=True).splitlines()]

    def four(nz):   # the rows' buffers of 72 complex per 128 points, and E1 and G0 of the strips for this one's modes
        return 4 * (nz // 128 * 72) * 8 + 2 * -(-nz // 128) * 128 * 4

    eight = 8 * (2048 // 128 * 72) * 8 + (3 * (512 + 512 // 32 + 1) + 2 * 32 * 64) * 4   # the r-line arrays too
    assert out == [(128, four(256)), (128, four(256)), (64, eight), (128, four(2048))]


MEMORY = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    for (int nr : {2, 32, 255, 1024}) {
        const size_t n = (size_t)nr * 256;
        std::vector<double> kappa(n, 1.0), q(n, 0.5);
        fake::mallocs.clear();
        axipcg_op_t op = nullptr;
        if (axipcg_op_create(nr, 256, 1, 1, 0, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
        for (size_t m : fake::mallocs) std::printf("%zu ", m);
        std::printf("\n");
        axipcg_op_destroy(op);
    }
    return 0;
}
"""


def test_reduced_factors_take_the_lanes_that_hold_strips(tmp_path_factory):
    """2 L + 13 values a mode and lane, of 1, 8 and 64 lanes of one strip (L = 1) and 64
    of four (L = 4), in both precisions: what the solves read and no more."""
    out = _hostcode.run(tmp_path_factory, MEMORY, library=True).splitlines()
    for line, (lanes, rows) in zip(out, ((1, 1), (8, 1), (64, 1), (64, 4))):
        sizes = [int(v) for v in line.split()]
        for width in (4, 8):
            assert 256 * (2 * rows + 13) * lanes * width in sizes
