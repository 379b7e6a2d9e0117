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
  while (std::scanf("%lld %lld %d", &B, &L, &d) == 3)
    std::printf("%d %d %d %d\\n", rom::scan_bwd_chunk(B, L, d), rom::scan_by_lane(B, L, d), rom::scan_by_lane(B, L, d, true),
                rom::scan_lane_chunks(B, L, d));
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


@pytest.mark.parametrize("B,L,d_inner,want", [
    (1, 8192, 768, 1), (1, 3900, 768, 0), (1, 2048, 1536, 1), (1, 1536, 1536, 0), (1, 3072, 2048, 1), (2, 1536, 1280, 1), (2, 1024, 1536, 0),
    (2, 3072, 2048, 0), (4, 1536, 1280, 1), (4, 1024, 1536, 0), (4, 3072, 1792, 1), (4, 3200, 2048, 1), (4, 1536, 2304, 1), (4, 1024, 2304, 0),
    (8, 2048, 1536, 0), (1, 6500, 4096, 1), (1, 600, 4096, 0), (1, 8192, 16, 0),
])
def test_lane_scan_of_few_blocks(rules, B, L, d_inner, want):
    """Both sides of the line for up to three workgroups per CU, where each was measured faster."""
    assert rules(B, L, d_inner)[1] == want


@pytest.mark.parametrize("B,L,d_inner,lane,chunks", [
    (1, 4500, 784, 0, None), (1, 5301, 784, 1, 165), (2, 1500, 1296, 1, 46), (1, 2999, 1040, 1, 93),        # chunks of 32 steps
])
def test_lane_scan_in_short_chunks(rules, B, L, d_inner, lane, chunks):
    """The shapes that test_gpu_scan_lane.py runs for them."""
    got = rules(B, L, d_inner)
    assert got[1] == lane and (chunks is None or got[3] == chunks)


@pytest.mark.parametrize("B,L,d_inner,want", [
    (1, 16384, 1536, 1), (1, 16383, 1536, 0), (2, 4096, 3072, 1), (4, 3000, 2048, 0), (4, 3072, 2048, 1), (8, 2048, 1536, 1),
    (1, 8192, 768, 0), (9, 4096, 1536, 0), (64, 256, 4096, 1), (1, 2048, 1536, 0),
])
def test_lane_scan_fp32(rules, B, L, d_inner, want):
    """24 Mi (step, channel) pairs at no more than three workgroups a CU, or enough wavefronts without chunks."""
    assert rules(B, L, d_inner)[2] == want


CHUNKS = r"""
#include <cstdio>
#include "rom_scan_rule.h"
int main() {
  for (long long B = 1; B < 40; B += 1 + B / 5)
    for (long long L = 1; L < 40000; L += 1 + L / 9)
      for (int d = 16; d < 6000; d += 16 * (1 + d / 100)) {
        const long long most = rom::scan_most_chunks(B, L, d), a = rom::scan_chunks(B, L, d), b = rom::scan_lane_chunks(B, L, d);
        if ((a > 1 && B * a > most) || (B * ((d + 63) / 64) < 2048 && b > 1 && B * b > most) || rom::scan_most_chunks(B + 1, L, d) < most ||
            rom::scan_most_chunks(B, L + 7, d) < most)
          return std::printf("%lld %lld %d\n", B, L, d), 1;
      }
  return 0;
}
"""


def test_chunk_states_fit_and_serve_smaller_calls(tmp_path):
    (tmp_path / "main.cpp").write_text(CHUNKS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "chunks")], check=True)
    r = subprocess.run([str(tmp_path / "chunks")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


ROOM = r"""
#include <cstdio>
#include "rom_scan_rule.h"
int main() {
  for (int f32 = 0; f32 < 2; ++f32)
    for (int d = 16; d < 6000; d += 16 * (1 + d / 60))
      for (long long B = 1; B < 900; B += 1 + B / 3) {
        long long shorter = 0;
        for (long long L = 1; L < 40000; L += 1 + L / 11) {
          const long long room = rom::scan_room_chunks(B, L, d, f32), a = rom::scan_chunks(B, L, d), lane = rom::scan_lane_chunks(B, L, d);
          const long long used = rom::scan_by_lane(B, L, d, f32) && lane > 1 ? B * lane : a > 1 ? B * a : 0;
          if (used > room || room < shorter || rom::scan_room_chunks(B + 1, L, d, f32) < room || (L < 512 && room))
            return std::printf("%d %lld %lld %d\n", f32, B, L, d), 1;
          shorter = room;
        }
      }
  // calls that are not cut, and no smaller one is
  for (auto c : {std::array<int, 3>{64, 64, 4096}, {4, 511, 128}, {1, 2048, 4096}, {8, 1024, 4096}, {512, 500, 2048}})
    if (rom::scan_room_chunks(c[0], c[1], c[2], false)) return std::printf("room %d %d %d\n", c[0], c[1], c[2]), 1;
  return 0;
}
"""


def test_room_for_chunk_states(tmp_path):
    """What a call uses, no less for more or longer sequences, none where nothing is cut."""
    (tmp_path / "main.cpp").write_text("#include <array>\n#include <initializer_list>\n" + ROOM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "room")], check=True)
    r = subprocess.run([str(tmp_path / "room")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
