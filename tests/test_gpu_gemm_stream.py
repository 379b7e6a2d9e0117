"""The streamed routed GEMM.  Its last round, cut into 1, 2, 4 or 8 pieces a tile, and one whole tile per workgroup before it:
ragged and empty groups and column tiles, through the layer, the block (skip in the epilogue), the FFN-MoE layer (SwiGLU) and the
backward pass (contraction-major weights), against the oracle.  Workgroups that go on from tile to tile (more than two
rounds of 256 x 256 tiles, partial column tiles before and behind full ones, and the shortest inner dimensions it takes), for
each epilogue: against plain fp32 products of the call's own inputs."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomFfnMoe, RomLayer
from rom_synth import RomConfig, make_ffn_weights, make_input, make_weights
from gpu_util import BLOCK_EPS, TOL, check_rounded, compare_layer, grouped, rel_err, run_layer, to_np

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


@pytest.mark.parametrize("block", [False, True])
@pytest.mark.parametrize("N,E,d_model,d_inner,bias", [
    (30000, 3, 512, 544, None),                  # in projection 5 column tiles, 64 columns in the last
    (30000, 3, 576, 528, (9.0, 0.0, -9.0)),      # 32 in the last, an empty group
    (36000, 5, 832, 512, None),                  # out projection 4 column tiles, 64 in the last
    (48000, 4, 520, 512, (0.5, 0.0, 0.0, -9.0)), # 3 and 8
    (36000, 2, 320, 640, None), (36000, 3, 384, 528, None), (36000, 2, 448, 512, None),      # five, six and seven slabs
    (40000, 64, 576, 528, None), (36000, 5, 640, 704, None),      # as many groups as there are lanes; nine to eleven slabs
])
def test_stream_gemm_rounds(N, E, d_model, d_inner, bias, block):
    cfg = RomConfig(f"rounds_{N}", 860 + d_model % 97, 8, N // 8, d_model, d_inner, 16, 4, 32, E, 1, "bf16", 0, weight_std=0.05,
                    router_bias=bias)
    layer = RomLayer(cfg, make_weights(cfg))
    x = layer.to_device(make_input(cfg))
    out = layer.block_forward(x, eps=BLOCK_EPS) if block else layer.forward(x)
    xf = x.view(N, d_model)
    idx, gate = layer.ws_view("expert_idx", 8, N // 8)[:, 0], layer.ws_view("gate", 8, N // 8)
    w = layer.block_weights() if block else layer.weights
    xz = grouped(xf, w["w_in"], idx)
    if block:
        xz *= torch.rsqrt(xf.float().square().mean(-1, keepdim=True) + BLOCK_EPS)
    check_rounded(layer.ws_view("xz", 8, N // 8), xz)
    check_rounded(out.view(N, d_model), gate * grouped(layer.ws_view("g", 8, N // 8), w["w_out"], idx), xf if block else None)


def ffn_reference(x, ffn, idx, gate, pre_norm, skip):
    xin = x
    if pre_norm:
        xin = x * torch.rsqrt(x.square().mean(-1, keepdim=True) + BLOCK_EPS) * ffn.norm_w
    y = torch.zeros_like(x)
    for e in range(ffn.w_down.shape[0]):
        rows = (idx == e).nonzero().flatten()
        h = xin[rows] @ ffn.w_gate_up[e].float().T
        a = torch.nn.functional.silu(h[:, :ffn.d_ff]) * h[:, ffn.d_ff:]
        y = y.index_add(0, rows, gate[rows] * (a @ ffn.w_down[e].float().T))
    return x + y if skip else y


@pytest.mark.parametrize("pre_norm", [False, True])
@pytest.mark.parametrize("N,E,d_model,d_ff", [
    (30000, 3, 512, 544), (36000, 3, 832, 576), (30000, 5, 512, 1280), (36000, 2, 384, 1280), (36000, 2, 768, 320)])
def test_stream_gemm_rounds_ffn(N, E, d_model, d_ff, pre_norm):
    """SwiGLU and its row scale, the skip, and on the way back contraction-major weights, over several rounds."""
    cfg = RomConfig(f"rounds_ffn_{N}", 880 + d_ff % 89, 1, N, d_model, 64, 16, 4, 32, E, 1, "bf16", 0, weight_std=0.05)
    layer = RomLayer(cfg, make_weights(cfg))
    x = layer.to_device(make_input(cfg)).view(N, d_model)
    routing = layer.route(x)
    ffn = RomFfnMoe(layer, d_ff, make_ffn_weights(cfg, d_ff), eps=BLOCK_EPS)
    out = ffn.forward(x, routing, pre_norm=pre_norm, add_skip=pre_norm)
    d_out = layer.to_device(np.random.default_rng(N).standard_normal((N, d_model)).astype(np.float32))
    d_x, d_gate, grads = ffn.backward(x, routing, d_out, pre_norm=pre_norm, add_skip=pre_norm)
    xf = x.float().requires_grad_()
    gate = routing["gate"].clone().requires_grad_()
    ref = ffn_reference(xf, ffn, routing["expert_idx"][:, 0], gate, pre_norm, pre_norm)
    ref.backward(d_out.float())
    for name, got, want in (("out", out, ref.detach()), ("d_x", d_x, xf.grad), ("d_gate", d_gate, gate.grad)):
        err = ((got.float() - want).abs().max() / want.abs().max()).item()
        assert err <= TOL["bf16"], (name, err)
