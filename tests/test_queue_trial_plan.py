"""Which sizes of the FIFO and SORTED closed loop give every block a whole trial (queue_trial_plan.h), compiled for the host: points on both
sides of the line, as they were measured."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = """
#include <cstdio>
#include <cstdlib>
#include "queue_trial_plan.h"
int main(int, char** a) { printf("%d", queue_trials_pay(atoi(a[1]), atoi(a[2]))); }
"""


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    at = tmp_path_factory.mktemp("plan")
    (at / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_05906_amd", "csrc"), "-o", str(at / "plan"), str(at / "main.cpp")])
    return lambda n, b: bool(int(subprocess.check_output([str(at / "plan"), str(n), str(b)])))


@pytest.mark.parametrize("n,b,trials", [(100, 1, True), (129, 3, False), (129, 4, True), (512, 31, False), (512, 32, True), (513, 191, False), (513, 192, True), (4096, 256, True),
                                        # a second round of blocks
                                        (1000, 257, False), (1000, 300, False), (1000, 447, False), (1000, 448, True), (1000, 512, True), (1000, 700, True), (1000, 1024, False),
                                        (2000, 257, False), (2000, 500, True), (2500, 400, False), (4000, 257, False),
                                        # two trials to a compute unit
                                        (512, 257, False), (320, 300, False), (512, 448, True), (512, 512, True), (512, 513, False), (128, 1000, False)])
def test_line(pays, n, b, trials):
    assert pays(n, b) == trials
