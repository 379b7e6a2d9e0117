"""Where the conv's end state is written (rom_conv_rule.h, host code)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_18145_amd", "csrc")
MAIN = """
#include <cstdio>
#include "rom_conv_rule.h"
int main() {
  long long in, out, L, n;
  while (std::scanf("%lld %lld %lld %lld", &in, &out, &L, &n) == 4)
    std::printf("%d\\n", rom::conv_state_beside(reinterpret_cast<const float *>(in), reinterpret_cast<const float *>(out), L, n));
}
"""


@pytest.fixture(scope="module")
def beside(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "rule")], check=True)
    return lambda *a: subprocess.run([str(d / "rule")], input=" ".join(map(str, a)) + "\n", capture_output=True, text=True,
                                     check=True).stdout.strip() == "1"


# addresses in bytes, L, floats of state
@pytest.mark.parametrize("src,dst,L,n,want", [
    (4096, 8192, 33, 1024, False), (0, 8192, 33, 1024, False), (4096, 0, 33, 1024, False),      # apart, no old one, not wanted
    (4096, 4096, 33, 1024, True), (4096, 8176, 33, 1024, True), (8176, 4096, 33, 1024, True),   # the same, partly the same
    (4096, 4096, 32, 1024, False), (4096, 4096, 1, 1024, False),                                # one run reads before it writes
    (4096, 8196, 33, 1024, True), (0, 8200, 16384, 1024, True),                                 # no 16-byte stores
])
def test_state_beside(beside, src, dst, L, n, want):
    assert beside(src, dst, L, n) == want
