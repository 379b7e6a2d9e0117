"""Which selective scan takes a call and how the adjoint is cut into chunks (rom_scan_rule.h, host code): what was measured
fastest on either side of each line of the rules."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_18145_amd", "csrc")
MAIN = """
#include <cstdio>
#include "rom_scan_rule.h"
int main() {
  long long B, L; int d;
  while (std::scanf("%lld %lld %d", &B, &L, &d) == 3) std::printf("%d %d\\n", rom::scan_bwd_chunk(B, L, d), rom::scan_by_lane(B, L, d));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "rule")], check=True)

    def ask(*a):
        out = subprocess.run([str(d / "rule")], input=" ".join(map(str, a)) + "\n", capture_output=True, text=True, check=True)
        return [int(v) for v in out.stdout.split()]

    return ask


@pytest.mark.parametrize("B,L,d_inner,want", [
    (1, 16384, 4096, 128), (4, 2048, 2048, 128), (1, 2048, 2048, 128), (16, 64, 2048, 128), (64, 129, 2048, 128),
    (1, 1024, 2048, 32), (4, 300, 1536, 32), (1, 1000, 512, 32), (1, 4000, 128, 32),
    (2, 200, 512, 16), (1, 300, 64, 16), (1, 129, 128, 16), (1, 128, 512, 16), (1, 64, 128, 16),
    (8, 128, 2048, 128), (1, 16, 128, 128), (1, 32, 128, 128), (1, 1, 16, 128),
])
def test_adjoint_scan_chunks(rules, B, L, d_inner, want):
    assert rules(B, L, d_inner)[0] == want


@pytest.mark.parametrize("B,L,d_inner,want", [
    (64, 256, 4096, 1), (128, 2, 2048, 1), (64, 64, 2048, 1), (2048, 2, 64, 1), (8192, 40, 16, 1),
    (4096, 40, 16, 0), (2048, 40, 48, 0), (63, 256, 2048, 0),          # wavefronts with idle lanes do not count whole
    (1, 16384, 4096, 1), (2, 4096, 3072, 1), (4, 4096, 2048, 1), (4, 2048, 2048, 0), (8, 2048, 4096, 0), (1, 64, 128, 0),
])
def test_lane_scan(rules, B, L, d_inner, want):
    assert rules(B, L, d_inner)[1] == want
