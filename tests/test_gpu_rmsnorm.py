"""The adjoint of the RMS norm in one pass (rows of up to 2048 columns) and in two: rows that do not fill their pieces of 256 columns, rows
past a block's sixteen and blocks without any, through the FFN-MoE layer's backward against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomFfnMoe, RomLayer
from rom_synth import RomConfig, make_ffn_weights, make_input, make_weights
from gpu_util import BLOCK_EPS, TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d_model,dtype,skip", [
    (1, 8, "fp32", True), (3, 256, "fp32", True), (16, 264, "fp32", False), (17, 512, "bf16", True), (67, 520, "fp32", True),
    (130, 1032, "bf16", True), (35, 1544, "fp32", True), (50, 2048, "bf16", False), (50, 2048, "fp32", True), (33, 2056, "fp32", True),
    (8193, 16, "fp32", True),                                   # 17 rows a block, 30 blocks without any
])
def test_norm_backward(n, d_model, dtype, skip):
    cfg = RomConfig(f"rms_{n}", 700 + n % 89, 1, n, d_model, 64, 16, 4, 8, 2, 1, dtype, 0, weight_std=0.05)
    w, fw, x = make_weights(cfg), make_ffn_weights(cfg, 64), make_input(cfg)
    layer = RomLayer(cfg, w)
    xd = layer.to_device(x).view(n, d_model)
    routing = layer.route(xd)
    ffn = RomFfnMoe(layer, 64, fw, eps=BLOCK_EPS)
    ffn.forward(xd, routing, pre_norm=True, add_skip=skip)
    d_out = layer.to_device(np.random.default_rng(n).standard_normal((n, d_model)).astype(np.float32))
    d_x, _, grads = ffn.backward(xd, routing, d_out, pre_norm=True, add_skip=skip)
    torch.cuda.synchronize()
    ref = O.ffn_moe_backward(x.reshape(n, -1), fw["w_gate_up"], fw["w_down"], to_np(routing["expert_idx"]), to_np(routing["gate"]),
                             to_np(d_out), norm_w=fw["norm_w"], eps=BLOCK_EPS, skip=skip)
    assert rel_err(to_np(d_x).reshape(n, -1), ref["d_x"].reshape(n, -1)) <= TOL[dtype]
    assert rel_err(to_np(grads["d_norm_w"]), ref["d_norm_w"]) <= TOL[dtype]
