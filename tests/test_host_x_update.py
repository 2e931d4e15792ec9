"""The last x update of a PCG solve (x += alpha p by the inverse launch that finds
the solve stopped), as its own code decides it, on the host: only with a target,
in the iteration it belongs to, and with a step length to apply."""
from tests import _hostcode

DRIVER = r"""
#include <cstdio>
#include "wxform.h"
using namespace axipcg;
int main()
{
    double p[4] = {1, 2, 3, 4};
    PcgState st{};
    auto x0 = [&](XFin fin, double *x, double alpha, int cur) {
        for (int k = 0; k < 4; ++k) x[k] = 10;
        st.step = {alpha, cur, 0};
        for (int t = 0; t < 2; ++t) x_finish(fin, &st, 0, 4, t, 2);
        std::printf("%g %g %g %g\n", x[0], x[1], x[2], x[3]);
    };
    double x[4];
    x0(XFin{x, p, 3}, x, 0.5, 3);    // stopped in this launch's iteration
    x0(XFin{x, p, 3}, x, 0.5, 2);    // stopped in an earlier one
    x0(XFin{x, p, 0}, x, 0.0, 0);    // stopped at the start
    for (int cur = -1; cur < 2; ++cur) x0(XFin{}, x, 0.5, cur);   // no target
    return 0;
}
"""


def test_update_applies_in_its_own_iteration_and_with_a_target(tmp_path):
    still = "10 10 10 10"
    assert _hostcode.run(tmp_path, DRIVER).split("\n")[:6] == ["10.5 11 11.5 12", still, still, still, still, still]
