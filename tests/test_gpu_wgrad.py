"""The weight-gradient GEMM over outputs of whole 256 x 256 tiles, at the edges of its 64-position slabs and of the runs of 16
positions that a wavefront brings, of its patches of four tile rows, and with several tiles a workgroup; experts without
tokens among them.  Below 16 positions another kernel takes the call."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,d_model,d_inner,E,top_k,bias", [
    (15, 256, 512, 2, 1, None), (16, 256, 512, 2, 1, None), (17, 256, 256, 1, 1, None), (63, 768, 512, 3, 1, None),
    (64, 256, 1280, 1, 1, None), (65, 256, 512, 1, 1, None), (129, 512, 256, 4, 2, None),
    (200, 256, 512, 4, 1, (0.0, 9.0, -50.0, 0.0)), (100, 512, 512, 3, 1, (-50.0, -50.0, 0.0)),
    (90, 1024, 2048, 16, 1, None),                              # several tiles a workgroup, one slab each
    (700, 1024, 1536, 6, 1, None),                              # and two or three
])
def test_weight_gradients(L, d_model, d_inner, E, top_k, bias):
    cfg = RomConfig(f"wg_{L}", 800 + L % 97, 1, L, d_model, d_inner, 16, 4, 16, E, top_k, "bf16", int(top_k > 1), weight_std=0.05,
                    router_bias=bias)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    layer.forward(layer.to_device(x))
    idx = to_np(layer.ws_view("expert_idx", 1, L))
    d_out = layer.to_device(np.random.default_rng(L).standard_normal((1, L, d_model)).astype(np.float32))
    _, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    for name in ("d_w_in", "d_w_out"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name
        for e in range(E):                                      # an expert without tokens: zeros, not what was there
            if not (idx == e).any():
                assert not to_np(grads[name])[e].any()


@pytest.mark.parametrize("L,d_inner,rank,E,top_k,bias", [
    # dt_rank + 32 and dt_rank thin columns: two to five blocks of 32, whole and ragged, and past the last (136 + 32)
    (130, 144, 8, 2, 1, None), (320, 80, 32, 1, 1, None), (65, 272, 40, 1, 1, None), (193, 208, 64, 3, 1, (9.0, 0.0, -50.0)),
    (400, 64, 72, 2, 2, None), (257, 336, 96, 1, 1, None), (90, 144, 104, 4, 2, (0.0, 9.0, 9.0, -50.0)), (600, 400, 128, 2, 1, None),
    (1, 48, 136, 3, 1, None),
    # 128 wide columns a workgroup: one slab, and more than the ring holds
    (100, 4096, 24, 8, 1, None), (520, 4112, 128, 8, 1, (9.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, -50.0)),
])
def test_thin_weight_gradients(L, d_inner, rank, E, top_k, bias):
    cfg = RomConfig(f"wgt_{L}", 800 + L % 97, 1, L, 64, d_inner, 16, 4, rank, E, top_k, "bf16", int(top_k > 1), weight_std=0.05,
                    router_bias=bias)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    layer.forward(layer.to_device(x))
    idx = to_np(layer.ws_view("expert_idx", 1, L))
    d_out = layer.to_device(np.random.default_rng(L).standard_normal((1, L, 64)).astype(np.float32))
    _, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    for name in ("d_w_x", "d_w_dt"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name
        for e in range(E):
            if not (idx == e).any():
                assert not to_np(grads[name])[e].any()
