"""Which kernels route a call's tokens and group its slots (rom_route_rule.h, host code)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_18145_amd", "csrc")
MAIN = """
#include <cstdio>
#include "rom_route_rule.h"
int main() {
  int d, e;
  while (std::scanf("%d %d", &d, &e) == 2)
    std::printf("%lld %lld %d\\n", (long long)rom::route_four_most(d, e), (long long)rom::kRouteFewMost, rom::grouping_in_one(d, e));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "rule")], check=True)
    return lambda *a: [int(v) for v in subprocess.run([str(d / "rule")], input=" ".join(map(str, a)) + "\n", capture_output=True,
                                                      text=True, check=True).stdout.split()]


@pytest.mark.parametrize("d_model,n_experts,four", [
    (64, 8, 1024), (512, 16, 1024), (576, 8, 2304), (768, 8, 3072), (768, 4, 2048), (1024, 8, 4096), (1024, 6, 3072), (2048, 8, 4096),
    (1024, 1, 1024), (1024, 2, 2048), (2048, 2, 2048), (8192, 1, 4096), (640, 16, 3072), (2048, 16, 3072),
])
def test_four_wavefronts_for_a_token(rule, d_model, n_experts, four):
    """Both sides of the line as measured; never below what is too few for anything else."""
    assert rule(d_model, n_experts)[0] == four


def test_matrix_pipe_line(rule):
    """Its sums are less exact than the other kernels' (test_gpu_route.py holds theirs to a bound that it does not keep)."""
    assert rule(2048, 8)[1] == 8192


@pytest.mark.parametrize("n_slots,n_experts,one", [
    (1, 8, 1), (4096, 8, 1), (4097, 8, 0), (8192, 8, 0), (4096, 1, 1), (8192, 4, 0), (2048, 9, 1), (2049, 9, 0), (4096, 16, 0), (2048, 64, 1),
])
def test_grouping_in_one_workgroup(rule, n_slots, n_experts, one):
    """Up to where three launches are faster in a call."""
    assert rule(n_slots, n_experts)[2] == one
