"""The plan of the degree count (csrc/degree_plan.h), compiled by the host compiler: how
often an arc is read and how much memory the copies take, over the whole range of n."""
import os
import subprocess

import pytest

from paper_2507_11094_amd import build

CODE = r"""
#include <cstdio>
#include <cstdlib>
#include "degree_plan.h"
int main(int, char **a) {
    const long long n = atoll(a[1]), arcs = atoll(a[2]);
    int B = 1;
    while ((1ll << B) < n) ++B;
    const dg::DegreePlan p = dg::degree_plan(B, n, arcs);
    const int shift = B - p.part_bits;
    const long long reads = shift > DEG_RANGE_BITS ? 1ll << (shift - DEG_RANGE_BITS) : 1;
    printf("%d %d %d %lld\n", B, p.part_bits, p.copies, reads);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "p.cpp").write_text(CODE.replace("DEG_RANGE_BITS", "dg::DEG_RANGE_BITS"))
    subprocess.check_call(["g++", "-std=c++17", "-I", build.CSRC, str(d / "p.cpp"), "-o", str(d / "p")])
    return lambda n, arcs: [int(x) for x in subprocess.check_output([str(d / "p"), str(n), str(arcs)]).split()]


@pytest.mark.parametrize("n", [1, 2, 3, 255, 257, 1 << 13, 1 << 20, 1 << 21, (1 << 21) + 1, 1 << 22, 1 << 24,
                               (1 << 24) + 1, 1 << 26, 1 << 28, (1 << 29) + 1, 1 << 30])
@pytest.mark.parametrize("per", [0, 0.25, 1, 4, 16, 100])
def test_plan(plan, n, per):
    arcs = int(min(n * per, (1 << 31) - 1))
    B, part_bits, copies, reads = plan(n, arcs)
    assert 1 <= part_bits <= B
    passes = -(-part_bits // 8)
    # a pass of the sort costs about six reads of the keys; the sort of the whole arcs that
    # gave the degrees before took 2 B / 8 passes
    assert reads <= 8 and 6 * passes + reads <= 14
    assert passes * 6 + reads <= 6 * max(2 * B // 8, 2) + 6
    # no more than the row starts, or the entries with their weights, of the built graph
    assert 1 <= copies <= 8 and 4 * copies * n <= max(8 * n, 8 * arcs)
