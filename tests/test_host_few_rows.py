"""Few rows that strips of four do not divide run per mode unless the strips were set:
standalone applies up to 64 rows, solves at even counts up to 64."""
from tests import _hostcode

DRIVER = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    for (int nr : {2, 33, 60, 62, 63, 64, 65, 66})
        for (int set = 0; set < 2; ++set)
            for (int prec : {AXIPCG_PREC_FP64, AXIPCG_PREC_FP32}) {
                const size_t n = (size_t)nr * 1024;
                std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
                axipcg_op_t op = nullptr;
                if (axipcg_op_create(nr, 1024, 1, 1, 1, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
                if (set) axipcg_op_set_strips(op, 1);
                auto strips = [&] {
                    int s = 0, m = 0;
                    for (const fake::Launch &l : fake::launches) {
                        s += fake::has(l.kernel, "k_strip_");
                        m += fake::has(l.kernel, "k_tridiag");
                    }
                    return s && m ? -1 : s > 0;
                };
                fake::launches.clear();
                if (axipcg_precond_apply(op, b.data(), x.data(), prec, nullptr)) return 3;
                const int apply = strips();
                fake::launches.clear();
                if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 1, prec, 0, nullptr, nullptr) < 0) return 4;
                const int solve = strips();
                int active = 0;
                axipcg_op_strips_info(op, prec, &active, nullptr);
                std::printf("%d %d %d %d %d\n", nr, set, apply, solve, active);
                axipcg_op_destroy(op);
            }
    return 0;
}
"""


def test_few_rows(tmp_path_factory):
    lines = _hostcode.run(tmp_path_factory, DRIVER, library=True).splitlines()
    assert len(lines) == 32
    for line in lines:
        nr, were_set, apply, solve, active = map(int, line.split())
        few = nr % 4 != 0 and nr <= 64 and not were_set
        assert (apply, solve) == (int(not few), int(not (few and nr % 2 == 0))), line
        assert active == solve
