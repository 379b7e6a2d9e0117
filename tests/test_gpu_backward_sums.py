"""The backward's small reductions at the edges of their tiles: conv runs of 16 and 32 steps with ragged ends (64 and 128 are
cfg1's and cfg2's), the router's rounds of 64 and 16 tokens and both its chunk lengths, weight gradients of the x and dt projections
in 64 x 64 and 128 x 128 tiles that the output does not fill, experts without tokens."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d_model,d_inner,rank,E,dtype,bias", [
    # (one token in fp32: its gradients are single products, whose operands carry the bf16 roundings of all stages in front, up to
    # eight of 2^-8 that nothing averages, over 2e-2)
    (1, 1, 8, 16, 8, 2, "fp32", None), (2, 16, 512, 32, 8, 9, "fp32", None), (1, 17, 520, 48, 8, 3, "fp32", None),
    (3, 33, 1032, 144, 16, 17, "fp32", None), (1, 63, 24, 80, 8, 4, "bf16", None), (1, 65, 16, 64, 32, 2, "bf16", None),
    (2, 79, 64, 208, 40, 3, "bf16", (0.0, -50.0, 0.0)),         # 72 and 40 outputs
    (1, 129, 64, 272, 104, 5, "bf16", None), (1, 70, 32, 4096, 128, 8, "bf16", None), (2, 65, 32, 4112, 136, 8, "bf16", None),
    (64, 130, 32, 1600, 8, 4, "fp32", None),
])
def test_backward_sums(B, L, d_model, d_inner, rank, E, dtype, bias):
    cfg = RomConfig(f"sum_{L}", 600 + L % 97, B, L, d_model, d_inner, 16, 4, rank, E, 1, dtype, 0, weight_std=0.1, router_bias=bias)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    layer.forward(layer.to_device(x))
    idx = to_np(layer.ws_view("expert_idx", B, L))
    d_out = layer.to_device(np.random.default_rng(L).standard_normal((B, L, d_model)).astype(np.float32))
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL[dtype]
    for name in grads:
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL[dtype], name
