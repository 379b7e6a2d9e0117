"""The streamed routed GEMM: ragged and empty groups, ragged column tiles, and token counts that leave its last round cut
into 1, 2, 4 or 8 pieces a tile, through the layer, the block (skip in the epilogue), the FFN-MoE layer (SwiGLU) and the
backward pass (contraction-major weights)."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomFfnMoe
from rom_synth import RomConfig, make_ffn_weights
from gpu_util import BLOCK_EPS, TOL, compare_layer, rel_err, run_layer, to_np

pytestmark = pytest.mark.gpu


def cfg_of(L, E=2, K=1, d_model=576, d_inner=1088, bias=None, B=1):
    return RomConfig(f"stream_{L}", 800 + L % 97, B, L, d_model, d_inner, 16, 4, 32, E, K, "bf16", K > 1, weight_std=0.05,
                     router_bias=bias)


@pytest.mark.parametrize("kw", [
    dict(L=800), dict(L=1100), dict(L=2050), dict(L=3001), dict(L=6100), dict(L=9000, E=5), dict(L=1500, E=3, bias=(9.0, 0.0, -9.0)),
    dict(L=1024, E=4, K=2), dict(L=770, E=1),
])
@pytest.mark.parametrize("block", [False, True])
def test_stream_gemm_layer(kw, block):
    cfg = cfg_of(**kw)
    _, gpu, x, w = run_layer(cfg, block=block)
    compare_layer(cfg, gpu, x, w, block=block)


@pytest.mark.parametrize("L,d_ff", [(900, 544), (2100, 1088), (5000, 800)])
def test_stream_gemm_ffn(L, d_ff):
    cfg = cfg_of(L, E=2)
    layer, gpu, x, w = run_layer(cfg)
    fw = make_ffn_weights(cfg, d_ff)
    routing = {n: layer.ws_view(n, 1, L).clone() for n in ("offsets", "perm", "inv_perm", "gate")}
    out = RomFfnMoe(layer, d_ff, fw).forward(layer.to_device(x), routing, pre_norm=True, add_skip=True)
    ref = O.ffn_moe_forward(x.reshape(L, -1), fw["w_gate_up"], fw["w_down"], gpu["expert_idx"], gpu["gate"], norm_w=fw["norm_w"],
                            eps=BLOCK_EPS, skip=True)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert rel_err(to_np(out).reshape(L, -1), np.asarray(ref).reshape(L, -1)) <= TOL["bf16"]


@pytest.mark.parametrize("L,E", [(900, 2), (2300, 2), (1200, 3)])
def test_stream_gemm_backward(L, E):
    cfg = cfg_of(L, E=E, d_model=512, d_inner=1024)
    layer, gpu, x, w = run_layer(cfg)
    d_out = np.random.default_rng(L).standard_normal((1, L, 512)).astype(np.float32)
    d_out = layer.to_device(d_out)
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=gpu["expert_idx"])
    torch.cuda.synchronize()
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL["bf16"]
    for name in ("d_w_in", "d_w_out", "d_w_x", "d_w_dt", "d_A_log", "d_w_router"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name
