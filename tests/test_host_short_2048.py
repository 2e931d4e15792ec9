"""The form of FP32 solves on few rows of 2048 points follows the handle's switches as
they stand: strips where they were set or where single launches are on and can serve
the row count, the block-wide form otherwise."""
from tests import _hostcode

DRIVER = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    for (int nr : {48, 57, 512, 513}) {
        const size_t n = (size_t)nr * 2048;
        std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
        axipcg_op_t op = nullptr;
        if (axipcg_op_create(nr, 2048, 1, 1, 0, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
        auto form = [&] {
            int active = 0, strips = 0, block = 0, strip = 0, one = 0;
            if (axipcg_op_strips_info(op, AXIPCG_PREC_FP32, &active, &strips)) std::printf("error ");
            fake::launches.clear();
            if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 1, AXIPCG_PREC_FP32, 0, nullptr, nullptr) < 0) std::printf("error ");
            for (const fake::Launch &l : fake::launches) {
                block += fake::has(l.kernel, "k_zfwd8");
                strip += fake::has(l.kernel, "k_strip_fwd");
                one += fake::has(l.kernel, "k_strip_one");
            }
            std::printf("%d/%d:%d%d%d ", active, strips, block, strip, one);   // forward launches: start and one step
        };
        form();
        axipcg_op_set_fused(op, 0);
        form();
        axipcg_op_set_fused(op, 1);
        form();
        axipcg_op_set_fused(op, 0);
        form();
        axipcg_op_set_strips(op, 1);
        form();
        std::printf("\n");
        axipcg_op_destroy(op);
    }
    return 0;
}
"""


def test_form_follows_the_switches(tmp_path_factory):
    out = _hostcode.run(tmp_path_factory, DRIVER, library=True).split("\n")
    wide = "0/0:200"
    for line, nr in zip(out, (48, 57, 512, 513)):
        strips = f"1/{-(-nr // 4)}:020"
        single = f"1/{nr // 4}:011" if nr % 4 == 0 else wide
        if nr > 512:
            assert line.split() == [strips] * 5
        else:
            assert line.split() == [wide, wide, single, wide, strips], nr


TRANSFORMS = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    for (int nr : {512, 640, 641, 2048}) {
        const size_t n = (size_t)nr * 2048;
        std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
        axipcg_op_t op = nullptr;
        if (axipcg_op_create(nr, 2048, 1, 1, 1, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
        axipcg_op_set_strips(op, 0);
        fake::launches.clear();
        if (axipcg_precond_apply(op, b.data(), x.data(), AXIPCG_PREC_FP32, nullptr)) return 3;
        if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 1, AXIPCG_PREC_FP32, 0, nullptr, nullptr) < 0) return 4;
        int wave = 0, block = 0, rows = 0;
        for (const fake::Launch &l : fake::launches) {
            if (fake::has(l.kernel, "k_zfwd_w<") || fake::has(l.kernel, "k_zinv_w<")) wave++;
            if (fake::has(l.kernel, "k_zfwd8<") || fake::has(l.kernel, "k_zinv8<")) {
                block++;
                rows += l.grid.x;
            }
        }
        std::printf("%d %d %d\n", wave, block, rows);
        axipcg_op_destroy(op);
    }
    return 0;
}
"""


def test_transforms_outside_strips(tmp_path_factory):
    """Block-wide with a row to a workgroup up to 640 rows of 2048 in FP32, one wave a row
    above (six transforms: an apply, a solve's start and one step)."""
    out = _hostcode.run(tmp_path_factory, TRANSFORMS, library=True).split("\n")
    assert out[:4] == [f"0 6 {6 * 512}", f"0 6 {6 * 640}", "6 0 0", "6 0 0"]
