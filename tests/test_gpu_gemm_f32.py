"""The fp32 routed GEMM (and the bf16 shapes that the bf16 kernels do not take) through the layer, against the oracle: inner
dimensions that end inside a 16-wide block, a group of 64 or a 16-byte piece, unaligned rows, one-row and empty groups, ragged
column tiles, stores of four columns and of single ones, and every form of the kernel: 16 x 16 and 32 x 32 products a wavefront, the
latter over a short and a long inner dimension, and through LDS where rows are read element by element."""
import pytest

from rom_synth import RomConfig
from gpu_util import compare_layer, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,d_model,d_inner,dt_rank,E,K,dtype,bias", [
    (1, 8, 16, 1, 3, 1, "fp32", None), (67, 40, 80, 5, 4, 2, "fp32", None), (64, 64, 128, 4, 4, 1, "fp32", None),
    (33, 72, 144, 7, 5, 1, "fp32", (9.0, 0.0, 0.0, 0.0, -9.0)), (300, 136, 272, 12, 2, 1, "fp32", None),
    (1000, 256, 528, 16, 2, 2, "fp32", None), (1900, 136, 272, 9, 3, 1, "fp32", None), (2300, 200, 272, 8, 3, 1, "fp32", None),
    (70, 64, 128, 5, 4, 1, "bf16", None), (1900, 136, 272, 9, 3, 1, "bf16", None),
    # 32 x 32 products over 264 (in projection)
    (1500, 264, 528, 8, 2, 1, "fp32", None),
    # dt projections: 32 x 32 products over 20, 68, 132 and 156
    (9000, 32, 1040, 20, 3, 1, "bf16", None), (2300, 32, 2064, 68, 2, 1, "fp32", None), (2300, 32, 2064, 132, 2, 1, "bf16", None),
    (2300, 32, 2064, 156, 4, 1, "fp32", (9.0, -50.0, 0.0, 0.0)),
    # through LDS: 9, 63 and 81
    (5000, 32, 528, 9, 2, 1, "bf16", None), (1300, 32, 2064, 63, 3, 1, "fp32", None), (1300, 32, 2064, 81, 2, 2, "bf16", None),
    # x projections of 45 columns, which leave stores of four out: bf16 rows read four at a time, small and sliced, and wide
    (40, 64, 1040, 13, 2, 1, "bf16", None), (17000, 32, 272, 13, 2, 1, "bf16", None),
])
def test_f32_gemm_layer(L, d_model, d_inner, dt_rank, E, K, dtype, bias):
    cfg = RomConfig(f"f32_{L}", 700 + L % 89, 1, L, d_model, d_inner, 16, 4, dt_rank, E, K, dtype, K > 1, weight_std=0.05,
                    router_bias=bias)
    _, gpu, x, w = run_layer(cfg)
    compare_layer(cfg, gpu, x, w)
