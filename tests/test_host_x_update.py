"""The last x update of a PCG solve (x += alpha p once the solve has stopped), on the
host: as its own code decides it, only with a target, in the iteration it belongs to
and with a step length to apply; and where it is launched."""
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


def test_update_applies_in_its_own_iteration_and_with_a_target(tmp_path_factory):
    still = "10 10 10 10"
    assert _hostcode.run(tmp_path_factory, DRIVER).split("\n")[:6] == ["10.5 11 11.5 12", still, still, still, still,
                                                                       still]


LAUNCHES = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    const int nr = 64, nz = 256, n = nr * nz;
    std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
    axipcg_op_t op = nullptr;
    if (axipcg_op_create(nr, nz, 1.0, 1.0, AXIPCG_Z_DIRICHLET, kappa.data(), q.data(), 0.0, -1.0, nullptr, &op)) return 2;
    for (int fused = 0; fused < 2; ++fused) {
        axipcg_op_set_fused(op, fused);
        fake::launches.clear();
        if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 3, AXIPCG_PREC_FP32, 0, nullptr, nullptr) < 0) return 3;
        int one = 0, inverse = 0, last = 0, after = 0;
        for (const fake::Launch &l : fake::launches) {
            if (fake::has(l.kernel, "k_pcg_last_x")) { last++; after = 0; }
            else after++;
            one += fake::has(l.kernel, "k_strip_one");
            inverse += fake::has(l.kernel, "k_strip_inv");
        }
        std::printf("%d %d %d %d\n", one, inverse, last, last ? after : 0);
    }
    return 0;
}
"""


def test_single_launches_leave_the_last_update_to_one_launch_at_the_end(tmp_path_factory):
    """A workgroup whose grid barrier gave up cannot know whether the others take its
    step for the last one, so the step itself must not touch x."""
    out = _hostcode.run(tmp_path_factory, LAUNCHES, library=True).split("\n")
    assert out[0] == "0 4 0 0"   # three launches: the inverse ones (with the start's) update x
    assert out[1] == "3 1 1 0"   # single launches: one update, after everything else
