"""The adjoint scan at the edges of its chunks (16, 32 and 128 steps), 16-step groups and 64-channel blocks."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d_inner,dtype,top_k", [
    (2, 1, 16, "fp32", 1), (1, 15, 80, "fp32", 1), (3, 17, 64, "fp32", 2), (1, 127, 48, "fp32", 1), (2, 128, 32, "bf16", 1),
    (2, 129, 144, "fp32", 1), (1, 300, 272, "fp32", 2), (2, 513, 96, "bf16", 1),
    (1, 33, 144, "fp32", 1), (2, 1000, 272, "bf16", 1), (1, 1025, 512, "fp32", 1),               # 16, 32, 32 steps
    (128, 129, 96, "fp32", 1), (64, 257, 176, "fp32", 1), (43, 300, 272, "bf16", 1), (256, 128, 80, "fp32", 2),      # 128 steps
])
def test_scan_backward(B, L, d_inner, dtype, top_k):
    cfg = RomConfig(f"sb_{L}", 700 + L % 97, B, L, 32, d_inner, 16, 4, 8, 4, top_k, dtype, int(top_k > 1), weight_std=0.1)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    layer.forward(layer.to_device(x))
    idx = to_np(layer.ws_view("expert_idx", B, L))
    d_out = layer.to_device(np.random.default_rng(L).standard_normal((B, L, cfg.d_model)).astype(np.float32))
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL[dtype]
    for name in grads:
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL[dtype], name


def test_rows_of_many_channels():
    """Rows whose byte pitch (z's and its gradient's are twice as wide) does not fit 24 bits."""
    cfg = RomConfig("sb_wide", 799, 1, 2, 8, (1 << 21) + 16, 16, 4, 8, 1, 1, "fp32", 0, weight_std=0.1)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    d_out = layer.to_device(np.random.default_rng(2).standard_normal((1, 2, 8)).astype(np.float32))
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=np.zeros((2, 1), np.int32))
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL["fp32"]
    for name in grads:
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["fp32"], name
