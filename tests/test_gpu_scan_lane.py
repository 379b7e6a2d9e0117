"""The lane = channel scan: calls with 2048 x 64 channels over all sequences or more (one pass), and few long sequences
(time chunks with a fold between the passes), at chunk remainders, a ragged last channel group and one long L."""
import numpy as np
import pytest

from rom_synth import RomConfig, make_states
from gpu_util import compare_layer, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d_inner,dtype", [
    (128, 2, 1024, "fp32"), (128, 7, 1040, "fp32"), (128, 8, 1040, "bf16"), (128, 9, 1040, "fp32"), (121, 19, 1088, "bf16"),
    (1, 25601, 1040, "fp32"), (3, 8200, 1040, "bf16"),
])
def test_scan_lane(B, L, d_inner, dtype):
    cfg = RomConfig(f"lane_{B}_{L}", 900 + L % 89, B, L, 64, d_inner, 16, 4, 8, 4, 1, dtype, 0)
    cs, ss = make_states(cfg)
    _, gpu, x, w = run_layer(cfg, cs, ss)
    assert np.isfinite(gpu["ssm_state"]).all()
    compare_layer(cfg, gpu, x, w, cs, ss)


@pytest.mark.parametrize("B,L,d_inner", [(1, 4500, 784), (1, 5301, 784), (2, 1500, 1296), (1, 2999, 1040)])
def test_scan_lane_short_chunks(B, L, d_inner):
    """Calls below 7 Mi (step, channel) pairs, whose chunks may be 32 steps long: remainders of chunks and of channel groups.  (The first lies
    just below the rule's line and takes lane = (channel, state); test_scan_rule.py holds which is which.)"""
    cfg = RomConfig(f"lane_short_{B}_{L}", 950 + L % 89, B, L, 64, d_inner, 16, 4, 8, 4, 1, "bf16", 0)
    cs, ss = make_states(cfg)
    _, gpu, x, w = run_layer(cfg, cs, ss)
    assert np.isfinite(gpu["ssm_state"]).all()
    compare_layer(cfg, gpu, x, w, cs, ss)
