"""The routed GEMM of a few rows (at most 8 positions, and 9 beside it): one group and many, empty groups, inner
dimensions that leave wavefronts without a unit, both tile widths with ragged column tiles (8 mod 16 columns, 16 mod 32), calls that
go back to the tiled kernel (short inner dimension, many workgroups), and every epilogue: plain, row scale (layer), row scale
and skip (block), per-slot rows (top-2), partial sums (x projection), SwiGLU (FFN-MoE)."""
import numpy as np
import pytest

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomFfnMoe, RomGdnLayer, RomMamba2Layer
from rom_synth import (RomConfig, get_gdn_config, get_mamba2_config, make_ffn_weights, make_gdn_input, make_gdn_weights,
                       make_mamba2_input, make_mamba2_weights)
from gpu_util import BLOCK_EPS, TOL, check_rounded, compare_layer, grouped, rel_err, run_layer, to_np

pytestmark = pytest.mark.gpu


def cfg_of(L, E=3, K=1, d_model=576, d_inner=1088, bias=None, B=1):
    return RomConfig(f"few_{L}", 500 + L, B, L, d_model, d_inner, 16, 4, 32, E, K, "bf16", True, weight_std=0.05, router_bias=bias)


@pytest.mark.parametrize("kw", [
    dict(L=2), dict(L=7, E=1), dict(L=8), dict(L=9), dict(L=8, E=1), dict(L=5, bias=(9.0, 0.0, -9.0)), dict(L=4, E=8, K=2),
    dict(L=3, E=5, K=2), dict(L=8, E=64), dict(L=8, E=2, bias=(-9.0, 9.0)), dict(L=6, d_inner=2112),
    dict(L=8, d_model=2048, d_inner=4096, E=2), dict(L=1, B=5, d_model=64, d_inner=128), dict(L=3, d_inner=1104),
    dict(L=5, d_model=584), dict(L=8, E=1, d_model=584, d_inner=2112), dict(L=7, d_model=1032, E=4),      # 8 mod 16 outputs
    dict(L=8, E=8, d_model=1024, d_inner=2048), dict(L=6, E=24, d_model=1024, d_inner=1536),
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


@pytest.mark.parametrize("n", [1, 3, 8])
@pytest.mark.parametrize("kind", ["gdn", "mamba2"])
def test_few_rows_ragged_wide_tiles(kind, n):
    """Input projections of 16 mod 32 columns (two outputs per head behind the wide parts): the last 32-wide tile is half there."""
    if kind == "gdn":
        cfg = get_gdn_config("gdn_small", cfg_id=91, batch=n, seq_len=1, d_model=1536, n_heads=24)
        layer, x, name, src = RomGdnLayer(cfg, make_gdn_weights(cfg)), make_gdn_input(cfg), "proj", "y"
    else:
        cfg = get_mamba2_config("m2_small", cfg_id=92, batch=n, seq_len=1, d_model=1536, d_inner=3072, d_state=128)
        layer, x, name, src = RomMamba2Layer(cfg, make_mamba2_weights(cfg)), make_mamba2_input(cfg), "zxbcdt", "g"
    assert cfg.d_in_proj % 32 == 16 and cfg.d_in_proj > 4096
    x = layer.to_device(x)
    out = layer.forward(x)
    idx, gate = layer.ws_view("expert_idx", n, 1)[:, 0], layer.ws_view("gate", n, 1)
    check_rounded(layer.ws_view(name, n, 1), grouped(x.view(n, -1), layer.weights["w_in"], idx))
    check_rounded(out.view(n, -1), gate * grouped(layer.ws_view(src, n, 1), layer.weights["w_out"], idx))
