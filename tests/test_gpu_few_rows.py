"""The routed GEMM of a few rows (at most 8 positions, and 9 beside it): one group and many, empty groups, inner
dimensions that leave wavefronts without a unit, ragged column tiles, both tile widths, and every epilogue: plain, row scale
(layer), row scale and skip (block), per-slot rows (top-2), partial sums (x projection), SwiGLU (FFN-MoE)."""
import numpy as np
import pytest

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomFfnMoe
from rom_synth import RomConfig, make_ffn_weights
from gpu_util import BLOCK_EPS, TOL, compare_layer, rel_err, run_layer, to_np

pytestmark = pytest.mark.gpu


def cfg_of(L, E=3, K=1, d_model=576, d_inner=1104, bias=None, B=1):
    return RomConfig(f"few_{L}", 500 + L, B, L, d_model, d_inner, 16, 4, 32, E, K, "bf16", True, weight_std=0.05, router_bias=bias)


@pytest.mark.parametrize("kw", [
    dict(L=2), dict(L=7, E=1), dict(L=8), dict(L=9), dict(L=8, E=1), dict(L=5, bias=(9.0, 0.0, -9.0)), dict(L=4, E=8, K=2),
    dict(L=3, E=5, K=2), dict(L=8, E=64), dict(L=8, E=2, bias=(-9.0, 9.0)), dict(L=6, d_inner=2112),
    dict(L=8, d_model=2048, d_inner=4096, E=2), dict(L=1, B=5, d_model=64, d_inner=128),
])
@pytest.mark.parametrize("block", [False, True])
def test_few_rows_layer(kw, block):
    cfg = cfg_of(**kw)
    _, gpu, x, w = run_layer(cfg, block=block)
    compare_layer(cfg, gpu, x, w, block=block)


@pytest.mark.parametrize("L,d_ff", [(1, 544), (5, 1088), (8, 2112)])
@pytest.mark.parametrize("pre_norm", [False, True])
def test_few_rows_ffn(L, d_ff, pre_norm):
    cfg = cfg_of(L)
    layer, gpu, x, w = run_layer(cfg)
    fw = make_ffn_weights(cfg, d_ff)
    routing = {n: layer.ws_view(n, 1, L).clone() for n in ("offsets", "perm", "inv_perm", "gate")}
    out = RomFfnMoe(layer, d_ff, fw).forward(layer.to_device(x), routing, pre_norm=pre_norm, add_skip=pre_norm)
    ref = O.ffn_moe_forward(x.reshape(L, -1), fw["w_gate_up"], fw["w_down"], gpu["expert_idx"], gpu["gate"],
                            norm_w=fw["norm_w"] if pre_norm else None, eps=BLOCK_EPS, skip=pre_norm)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert rel_err(to_np(out).reshape(L, -1), np.asarray(ref).reshape(L, -1)) <= TOL["bf16"]
