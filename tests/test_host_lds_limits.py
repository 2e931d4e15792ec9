"""A kernel's limit of dynamic LDS belongs to the device that is current when it is
set: on every device that a process uses, each launch above the default 64 KiB has
its limit raised there, whichever device came first.  Forms that go above it: the
one-workgroup solve, 8-row strips on long lines, the per-mode r-solve on long lines,
transforms of FP64 rows of 4096 points."""
from tests import _hostcode

DRIVER = r"""
#include <cstdio>
#include "_fake_hip.h"
#include "axipcg.h"
int main()
{
    struct Case { int nr, nz, strips; };
    const Case cases[] = {{64, 64, 1}, {256, 16, 1}, {31, 128, 1}, {4096, 256, 8}, {4000, 32, 1}, {4, 4096, 1}};
    for (int dev : {1, 0, 1, 2})
        for (const Case &c : cases)
            for (int prec : {AXIPCG_PREC_FP64, AXIPCG_PREC_FP32}) {
                fake::device = dev;
                const size_t n = (size_t)c.nr * c.nz;
                std::vector<double> kappa(n, 1.0), q(n, 0.5), b(n, 1.0), x(n, 0.0);
                axipcg_op_t op = nullptr;
                if (axipcg_op_create(c.nr, c.nz, 1, 1, AXIPCG_Z_NEUMANN, kappa.data(), q.data(), 0, -1, nullptr, &op)) return 2;
                axipcg_op_set_strips(op, c.strips);
                if (axipcg_pcg_solve(op, b.data(), x.data(), 1e-10, 1, prec, 0, nullptr, nullptr) < 0) return 3;
                if (axipcg_precond_apply(op, b.data(), x.data(), prec, nullptr)) return 4;
                axipcg_op_destroy(op);
            }
    int big = 0;
    for (const fake::Launch &l : fake::launches) {
        if (l.lds <= 65536) continue;
        big++;
        bool raised = false;
        for (const fake::Limit &m : fake::limits)
            raised |= m.kernel == l.kernel && m.device == l.device && (size_t)m.bytes >= l.lds;
        if (!raised) {
            std::printf("device %d, %zu bytes, no limit: %s\n", l.device, l.lds, l.kernel.c_str());
            return 1;
        }
    }
    std::printf("%d\n", big);
    return 0;
}
"""


def test_limits_are_raised_on_every_device(tmp_path_factory):
    assert int(_hostcode.run(tmp_path_factory, DRIVER, library=True)) >= 40
