"""The rule that sends a reverse sweep to k_bwd_trial (reverse_trial_plan.h), compiled for the host: what fits LDS, and that networks whose
row positions need more than the kernel's 32 bits are left to the other kernels."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = """
#include <cstdio>
#include <cstdlib>
#include "reverse_trial_plan.h"
int main(int, char** a) {
  const int N = atoi(a[1]), d_max = atoi(a[4]);
  const RevTrialPlan p = rev_trial_plan(N, atoi(a[2]), atoll(a[3]), d_max);
  printf("%d %d %d", p.H, p.P, p.P == 0 || rev_trial_fixed(N, p.P) + 4LL * p.H * N <= kRevTrialLds);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    at = tmp_path_factory.mktemp("plan")
    (at / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_05906_amd", "csrc"), "-o", str(at / "plan"), str(at / "main.cpp")])
    return lambda *args: [int(x) for x in subprocess.check_output([str(at / "plan")] + [str(x) for x in args]).split()]


def test_rows_beyond_32_bits_are_left_to_the_other_kernels(plan):
    for n, d_max in ((1, 5), (1000, 50), (1024, 120)):
        assert plan(n, 1, 2**31 - 1, d_max)[1] > 0
        for s in (2**31, 2**32, 2**32 + 100 * n, 2**40 - 1):
            assert plan(n, 1, s, d_max)[:2] == [0, 0]


@pytest.mark.parametrize("n,b,d_max,used", [(1, 1, 1, True), (100, 1, 20, True), (1000, 16, 50, True), (1000, 512, 50, True), (1024, 1, 120, True),
                                            (1025, 1, 50, False), (1000, 513, 50, False), (1024, 1, 250, False)])
def test_what_is_planned_fits(plan, n, b, d_max, used):
    H, P, fits = plan(n, b, 100 * n, d_max)
    assert fits and (P > 0) == used
    if used:
        assert 1 <= H <= d_max <= H * P and (P - 1) * H < d_max
