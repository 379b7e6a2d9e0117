"""The fp32 routed GEMM (and the bf16 shapes that the bf16 kernels do not take) through the layer, against the oracle: inner
dimensions that end inside a 16-wide block, a group of 64 or a 16-byte piece, unaligned rows, one-row and empty groups, ragged
column tiles, on either side of the line between 16 x 16 and 32 x 32 products a wavefront."""
import pytest

from rom_synth import RomConfig
from gpu_util import compare_layer, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,d_model,d_inner,dt_rank,E,K,dtype,bias", [
    (1, 8, 16, 1, 3, 1, "fp32", None), (67, 40, 80, 5, 4, 2, "fp32", None), (64, 64, 128, 4, 4, 1, "fp32", None),
    (33, 72, 144, 7, 5, 1, "fp32", (9.0, 0.0, 0.0, 0.0, -9.0)), (300, 136, 272, 12, 2, 1, "fp32", None),
    (1000, 256, 528, 16, 2, 2, "fp32", None), (1900, 136, 272, 9, 3, 1, "fp32", None), (2300, 200, 272, 8, 3, 1, "fp32", None),
    (70, 64, 128, 5, 4, 1, "bf16", None), (1900, 136, 272, 9, 3, 1, "bf16", None),
])
def test_f32_gemm_layer(L, d_model, d_inner, dt_rank, E, K, dtype, bias):
    cfg = RomConfig(f"f32_{L}", 700 + L % 89, 1, L, d_model, d_inner, 16, 4, dt_rank, E, K, dtype, K > 1, weight_std=0.05,
                    router_bias=bias)
    _, gpu, x, w = run_layer(cfg)
    compare_layer(cfg, gpu, x, w)
