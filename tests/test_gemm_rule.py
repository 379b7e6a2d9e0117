"""Which tile kernel a routed GEMM takes (rom_gemm_rule.h, host code): the kernel measured fastest on either side of each line
of the rule, and what the kernels cannot do."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_18145_amd", "csrc")
NAMES = ("stream", "dma256", "reg256", "t128", "skinny")
F32_NAMES = ("small", "wide", "wide_short", "staged")
MAIN = """
#include <cstdio>
#include "rom_gemm_rule.h"
int main() {
  long long M; int g, N, K, dma, wide, km, ip, f;
  while (std::scanf("%lld %d %d %d %d %d %d %d %d", &M, &g, &N, &K, &dma, &wide, &km, &ip, &f) == 9)
    std::printf("%d %d %d\\n", static_cast<int>(rom::gemm_tile({M, g, N, K, dma != 0, wide != 0, km != 0, ip != 0, f != 0})),
                rom::gemm_few_rows(M, g, N, K), static_cast<int>(rom::gemm_f32_tile(M, g, N, K, 1, wide == 0)));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "rule")], check=True)

    def ask(M, groups, N, K, dma=None, wide=False, w_kmajor=False, in_place=False, f32_or_softplus=False):
        dma = (K % 64 == 0 and not wide) if dma is None else dma
        line = " ".join(str(int(v)) for v in (M, groups, N, K, dma, wide, w_kmajor, in_place, f32_or_softplus))
        out = subprocess.run([str(d / "rule")], input=line + "\n", capture_output=True, text=True, check=True).stdout
        which, few, f32 = out.split()
        return NAMES[int(which)], few == "1", F32_NAMES[int(f32)]

    return ask


@pytest.fixture(scope="module")
def tile(rule):
    return lambda *a, **k: rule(*a, **k)[0]


@pytest.mark.parametrize("M,groups,N,K,want", [
    (16384, 8, 8192, 2048, "stream"), (16384, 8, 2048, 4096, "stream"), (16384, 8, 4096, 1024, "stream"),
    (16384, 8, 1024, 2048, "stream"), (1024, 8, 8192, 2048, "stream"), (7664, 8, 1024, 1536, "stream"), (2476, 4, 256, 640, "stream"),
    (16384, 8, 1536, 448, "stream"), (16384, 8, 2048, 512, "stream"),
    # slower as a stream of big tiles: a partial round in quarters, in halves over a short K, mostly padding
    (3072, 8, 1024, 2048, "t128"), (1536, 4, 2048, 4096, "t128"), (768, 2, 2048, 4096, "t128"), (5387, 8, 1024, 768, "t128"),
    (400, 1, 1024, 2048, "t128"), (512, 1, 8192, 2048, "t128"), (400, 1, 8192, 2048, "t128"),
    (14736, 16, 384, 1536, "t128"), (23704, 8, 640, 384, "t128"),
    # few rows a group
    (2720, 16, 3072, 768, "t128"), (2800, 16, 1536, 3072, "t128"), (2720, 16, 8192, 2048, "stream"),
    # no whole slabs
    (16384, 8, 4000, 1000, "t128"), (16384, 8, 2080, 520, "t128"),
    # as many groups as there are lanes (the entry points take no more)
    (40000, 64, 8192, 2048, "stream"),
    # the recurrent step
    (256, 8, 8192, 2048, "skinny"),
])
def test_measured_shapes(tile, M, groups, N, K, want):
    assert tile(M, groups, N, K) == want


def test_wide_activations_keep_the_big_tile(tile):
    assert tile(524288, 8, 2048, 4096, wide=True) == "reg256"


@pytest.mark.parametrize("K", [320, 384, 448, 512, 2048])
@pytest.mark.parametrize("M", [4096, 16384])
def test_contraction_major_weights_are_not_transposed(tile, M, K):
    assert tile(M, 4, 1536, K, w_kmajor=True) == "stream"


def test_fp32_and_softplus_epilogues(tile):
    assert tile(16384, 8, 4096, 512, f32_or_softplus=True) == "dma256"
    assert tile(15373, 4, 1024, 768, f32_or_softplus=True) == "dma256"
    assert tile(16695, 4, 1024, 1536, f32_or_softplus=True) == "t128"
    assert tile(4096, 1, 256, 4096, f32_or_softplus=True) == "t128"
    assert tile(16384, 8, 4096, 512, dma=False, f32_or_softplus=True) == "t128"


def test_what_the_stream_kernel_cannot_do(tile):
    big = dict(M=16384, groups=8, N=2048)
    assert tile(K=256, **big) == "t128"                              # its schedule needs five slabs
    assert tile(K=2048, dma=False, **big) == "t128"
    assert tile(K=2048, in_place=True, **big) == "t128"              # rows past a group's end are stored twice
    assert tile(M=1 << 30, groups=8, N=2048, K=512) == "t128"        # 32-bit positions


@pytest.mark.parametrize("M,groups,N,K,want", [
    (1, 8, 8192, 2048, True), (8, 8, 8192, 2048, True), (8, 8, 2048, 4096, True), (8, 4, 3072, 1536, True), (9, 8, 8192, 2048, False),
    (1, 8, 4096, 1024, True), (8, 1, 4096, 1024, True), (8, 64, 4096, 1024, True),
    # as many workgroups as the CUs hold and a short inner dimension: the tiled kernel is faster
    (6, 8, 2048, 1024, False), (8, 8, 4096, 1024, False), (5, 16, 2048, 768, False), (8, 16, 1536, 768, False),
    (4, 8, 2048, 1000, False), (4, 65, 2048, 1024, False),              # no whole units, more groups than lanes
])
def test_few_rows(rule, M, groups, N, K, want):
    assert rule(M, groups, N, K)[1] == want


# fp32 operands and the bf16 shapes that no bf16 kernel takes: the form measured fastest on either side of each line
@pytest.mark.parametrize("M,N,K,vec,want", [
    (64, 8192, 2048, True, "small"), (256, 8192, 2048, True, "small"), (500, 4000, 1000, True, "small"),
    (256, 4800, 152, True, "small"), (512, 1680, 52, True, "small"), (1024, 1680, 52, True, "wide_short"),
    (8192, 4096, 256, True, "wide_short"), (8192, 4096, 260, True, "wide"),
    (512, 960, 2000, True, "small"), (512, 1000, 2000, True, "wide"), (8192, 8192, 2048, True, "wide"),
    (512, 2032, 63, False, "small"), (1024, 2032, 63, False, "staged"), (16384, 2032, 63, False, "staged"),
    (500, 6432, 201, False, "staged"), (64, 4848, 151, False, "small"),
])
def test_f32_gemm(rule, M, N, K, vec, want):
    assert rule(M, 8, N, K, wide=not vec)[2] == want


SMALLK = r"""
#include <initializer_list>
#include <cstdio>
#include "rom_gemm_rule.h"
int main() {
  for (int K = 1; K <= 200; ++K) {
    const bool step = K % 16 == 0 && K >= 32 && K <= 160, power = K == 32 || K == 64 || K == 128;
    for (long long M : {1ll, 767ll, 768ll, 100000ll})
      if (rom::gemm_smallk(M, 8, K, false) != (power || (step && M >= 768)) || rom::gemm_smallk(M, 8, K, true) != power)
        return std::printf("%d %lld\n", K, M), 1;
  }
  return 0;
}
"""


def test_short_contractions(tmp_path):
    """Every whole number of 16-wide steps from 32 to 160, not only the widths of some models."""
    (tmp_path / "main.cpp").write_text(SMALLK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "smallk")], check=True)
    r = subprocess.run([str(tmp_path / "smallk")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
