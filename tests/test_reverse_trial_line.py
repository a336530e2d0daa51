"""The line on a run's spikes up to which its reverse sweep goes by k_bwd_trial (reverse_trial_plan.h), compiled for the host: points on
both sides of it, as they were measured."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = """
#include <cstdio>
#include <cstdlib>
#include "reverse_trial_plan.h"
int main(int, char** a) {
  const int N = atoi(a[1]), B = atoi(a[3]);
  const long long S = atoll(a[2]) * N;
  const bool adm = atoi(a[5]);
  const RevTrialPlan p = rev_trial_plan(N, B, S, atoi(a[4]));
  printf("%d", p.P > 0 && atof(a[6]) * rev_trial_weight(S, N, p.P, adm) <= rev_trial_load(S, N, B, p.P, adm));
}
"""


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    at = tmp_path_factory.mktemp("line")
    (at / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_05906_amd", "csrc"), "-o", str(at / "line"), str(at / "main.cpp")])
    return lambda *args: bool(int(subprocess.check_output([str(at / "line")] + [str(int(x) if isinstance(x, bool) else x) for x in args])))


@pytest.mark.parametrize("n,row,b,d_max,adm,spikes,trials", [
    (128, 100, 512, 50, False, 2.0, False), (256, 100, 300, 50, False, 1.0, False), (128, 100, 257, 50, True, 0.3, False), (128, 100, 256, 50, False, 2.0, True),
    (128, 100, 1, 50, True, 1.0, True), (128, 100, 1, 50, True, 3.6, False), (128, 100, 2, 50, True, 8.0, False), (128, 100, 4, 50, True, 7.8, True),
    (256, 100, 4, 50, True, 1.0, True), (256, 100, 16, 50, True, 2.0, False), (256, 100, 64, 50, True, 4.0, True), (256, 100, 64, 50, True, 8.0, False),
    (128, 10, 1, 50, True, 7.3, True), (128, 10, 1, 50, True, 16.0, False), (256, 10, 2, 50, True, 16.0, True),
    (256, 100, 8, 50, False, 8.0, True), (256, 100, 8, 50, False, 16.0, False), (100, 10, 1, 20, False, 10.0, True), (1000, 100, 1, 50, False, 2.0, True)])
def test_line(chosen, n, row, b, d_max, adm, spikes, trials):
    assert chosen(n, row, b, d_max, adm, spikes) == trials
