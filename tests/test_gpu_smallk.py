"""The routed GEMM of a short inner dimension (32 to 160 in steps of 16), whose workgroups take equal runs of rows, through the layer's dt
projection (with activation, K = dt_rank) and what comes back through the x projection (without, K = dt_rank + 32, from 4096 rows and 1024
columns on): every K, both sides of the rule's line of 96 rows a group, several runs per group, uneven and empty groups, a ragged
last column slice; against plain fp32 products of the call's own inputs and the oracle."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, compare_layer, grouped, rel_err, run_layer, to_np

pytestmark = pytest.mark.gpu


def cfg_of(n, rank, d_inner, E, bias=None, B=1):
    return RomConfig(f"smallk_{n}_{rank}", 960 + rank % 31, B, n // B, 128, d_inner, 16, 4, rank, E, 1, "bf16", 0, router_bias=bias)


@pytest.mark.parametrize("rank", [16, 48, 80, 96, 112, 144, 160])       # (16: the general kernel)
@pytest.mark.parametrize("n,d_inner,E,bias", [
    (96 * 3 - 1, 208, 3, None), (96 * 3, 208, 3, None), (1500, 336, 5, (9.0, 0.0, 0.0, 0.0, -50.0)),
])
def test_smallk_layer(n, d_inner, E, bias, rank):
    cfg = cfg_of(n, rank, d_inner, E, bias)
    _, gpu, x, w = run_layer(cfg)
    compare_layer(cfg, gpu, x, w)


@pytest.mark.parametrize("n,rank,d_inner,E,bias", [
    (40000, 48, 1008, 8, None), (30000, 160, 528, 64, None), (50000, 80, 272, 6, (9.0, 0.0, 0.0, 3.0, 0.0, -50.0)),
    (20000, 96, 1104, 16, None), (24000, 112, 400, 8, None), (16000, 144, 656, 5, (9.0, 0.0, 0.0, 3.0, -50.0)), (40000, 32, 272, 3, None),
])
def test_smallk_runs(n, rank, d_inner, E, bias):
    """Many 32-row pieces to a run; the dt projection is softplus(dt_low W^T + b), rounded to bf16 (2^-8 of it, some ulps of the
    softplus' argument, and the fp32 sums' order)."""
    cfg = cfg_of(n, rank, d_inner, E, bias, B=8)
    layer = RomLayer(cfg, make_weights(cfg))
    layer.forward(layer.to_device(make_input(cfg)))
    idx = layer.ws_view("expert_idx", 8, n // 8)[:, 0]
    low = layer.ws_view("dt_low", 8, n // 8)
    y = grouped(low, layer.weights["w_dt"], idx) + layer.weights["dt_bias"].float()
    ref = torch.nn.functional.softplus(y, threshold=80.0)
    got = layer.ws_view("dt", 8, n // 8).float()
    bound = 2.0 ** -8 * ref * 1.01 + 2e-5 * (1 + y.abs()) * ref.clamp(max=1.0)
    assert ((got - ref).abs() / bound).max().item() <= 1.0


@pytest.mark.parametrize("n,rank,d_inner,E", [(700, 48, 336, 3), (900, 96, 272, 4), (1000, 160, 208, 2)])
def test_smallk_backward(n, rank, d_inner, E):
    cfg = cfg_of(n, rank, d_inner, E)
    layer, gpu, x, w = run_layer(cfg)
    d_out = layer.to_device(np.random.default_rng(n).standard_normal((1, n, 128)).astype(np.float32))
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=gpu["expert_idx"])
    torch.cuda.synchronize()
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL["bf16"]
    for name in ("d_w_in", "d_w_out", "d_w_x", "d_w_dt", "d_A_log", "d_w_router"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name


@pytest.mark.parametrize("rank", [16, 32, 48, 64, 80, 96, 112, 128])
@pytest.mark.parametrize("d_inner,E,bias", [(1024, 3, None), (1040, 6, (9.0, 0.0, 0.0, 3.0, 0.0, -50.0))])
def test_smallk_backward_many_rows(rank, d_inner, E, bias):
    """Past the line of the form without activation; its output goes through the conv's adjoint into these gradients."""
    n = 8 * 520
    cfg = cfg_of(n, rank, d_inner, E, bias, B=8)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    xd = layer.to_device(x)
    layer.forward(xd)
    idx = to_np(layer.ws_view("expert_idx", 8, n // 8))
    d_out = layer.to_device(np.random.default_rng(rank).standard_normal((8, n // 8, 128)).astype(np.float32))
    d_x, grads = layer.backward(xd, d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL["bf16"]
    for name in ("d_conv_w", "d_conv_b", "d_w_in", "d_w_x"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name
