"""Kernels that a rule of dispatch replaced are not built any more: the reduced systems
of 4-row strips with recomputed coefficients, more rows a lane than 512 strips of eight
rows need, and the Stockham transforms' forms for rows too long to keep twiddles in LDS."""
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
    assert reduced and all(re.match(r"k_strip_reduced<\w+, 8, [1248], \d>\(", n) for n in reduced), reduced
    assert sum(n.startswith("k_zfwd<") for n in names) == 2 * 2 * 3   # z condition, fused or not, FP32 and FP64 in one or two rows
