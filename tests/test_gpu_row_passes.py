"""The backward's row passes (rows scaled by their gate; the router's share of the input gradient), which give a row as many lanes as it
fills: rows narrower than a wavefront's 512 columns, whole and ragged, and wider; tokens that don't fill a wavefront's rows; against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model", [8, 24, 64, 72, 200, 256, 264, 512, 520, 1032])
@pytest.mark.parametrize("n,E,K,dtype", [(1, 2, 1, "fp32"), (37, 3, 1, "bf16"), (131, 9, 2, "fp32"), (66, 5, 2, "bf16")])
def test_row_passes(n, d_model, E, K, dtype):
    cfg = RomConfig(f"rows_{n}_{d_model}", 640 + d_model % 97, 1, n, d_model, 64, 16, 4, 8, E, K, dtype, int(K > 1), weight_std=0.05)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    xd = layer.to_device(x)
    layer.forward(xd)
    idx = to_np(layer.ws_view("expert_idx", 1, n))
    # gate gradients of the size that makes the router's share of d_x count
    d_out = layer.to_device(np.random.default_rng(n).standard_normal((1, n, d_model)).astype(np.float32) * 4)
    d_x, grads = layer.backward(xd, d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL[dtype]
    for name in ("d_w_out", "d_w_router"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL[dtype], name
