"""The short conv: runs of one batch and of several, ragged sequence ends, a carried state from and to memory of its own and
in place, against the formula on the layer's own xz in fp32."""
import pytest
import torch

from paper_2506_18145_amd import RomLayer, RomMamba2Layer
from paper_2506_18145_amd.binding import rom_layer_forward, rom_mamba2_forward
from rom_synth import RomConfig, get_mamba2_config, make_input, make_mamba2_input, make_mamba2_weights, make_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("B,L,d_inner", [
    (3, 1, 48), (2, 2, 80), (1, 3, 48), (2, 7, 48), (2, 8, 272), (1, 9, 48), (2, 31, 80), (3, 32, 48), (2, 33, 80), (1, 70, 272),
    (1, 32771, 512),                                           # long runs, the last one ragged
])
def test_conv(B, L, d_inner, dtype):
    cfg = RomConfig(f"conv_{L}", 700 + L % 89, B, L, 64, d_inner, 16, 4, 8, 2, 1, dtype, 0, weight_std=0.05)
    layer = RomLayer(cfg, make_weights(cfg))
    x = layer.to_device(make_input(cfg))
    gen = torch.Generator(device="cuda").manual_seed(L)
    before = torch.randn(B, d_inner, 3, generator=gen, device="cuda")
    ssm = torch.randn(B, d_inner, 16, generator=gen, device="cuda")
    _, after, ssm_after = layer.forward(x, before, ssm, return_states=True)
    u, xz = (layer.ws_view(n, B, L).clone() for n in ("u", "xz"))
    xs = xz.view(B, L, 2 * d_inner)[..., :d_inner].float()
    full = torch.cat([before.transpose(1, 2), xs], 1)          # [B, 3 + L, d_inner]
    w = layer.weights["conv_w"].float()
    c = sum(full[:, j:j + L] * w[:, j] for j in range(4)) + layer.weights["conv_b"].float()
    want = c * torch.sigmoid(c)
    # five roundings and the raw exp / reciprocal: within 16 ulp of the terms' size; bf16 adds half an ulp of the result
    bound = 16 * 2.0 ** -23 * (sum((full[:, j:j + L] * w[:, j]).abs() for j in range(4)) + 1) * (1 + c.abs())
    bound = bound + (2.0 ** -8 * want.abs() if dtype == "bf16" else 0)
    assert bool(((u.view(B, L, d_inner).float() - want).abs() <= bound).all())
    assert torch.equal(after, full[:, L:].transpose(1, 2))     # the last three inputs, exactly

    out = torch.empty_like(x)
    conv, state = before.clone(), ssm.clone()
    rom_layer_forward(layer.dims, layer.weights, x, B, L, conv, state, out, conv, state, layer.workspace(B, L))
    assert torch.equal(conv, after) and torch.equal(state, ssm_after) and torch.equal(layer.ws_view("u", B, L), u)


@pytest.mark.parametrize("kind,shift", [("layer", 1), ("layer", 3), ("layer", 240), ("mamba2", 240)])
def test_conv_state_places(kind, shift):
    """A longer call's end state where the conv cannot write it directly: not aligned to its stores, or on part of the old one."""
    B, L = 2, 70
    if kind == "layer":
        cfg = RomConfig("conv_places", 790, B, L, 64, 80, 16, 4, 8, 2, 1, "bf16", 0, weight_std=0.05)
        layer, channels = RomLayer(cfg, make_weights(cfg)), 80
        call = lambda x, before, out, after, ws: rom_layer_forward(layer.dims, layer.weights, x, B, L, before, None, out, after, None, ws)
    else:
        cfg = get_mamba2_config("m2_cfg2", batch=B, seq_len=L, d_model=256, d_inner=512)
        layer, channels = RomMamba2Layer(cfg, make_mamba2_weights(cfg)), cfg.d_conv_ch
        call = lambda x, before, out, after, ws: rom_mamba2_forward(layer.dims, layer.weights, x, B, L, 1e-5, before, None, out, after, None, ws)
    x = layer.to_device((make_input if kind == "layer" else make_mamba2_input)(cfg)).view(B, L, -1)
    n = B * channels * 3
    buf = torch.randn(2 * n + 16, generator=torch.Generator(device="cuda").manual_seed(shift), device="cuda")
    before, want, out, out2 = buf[:n].clone(), torch.empty(n, device="cuda"), torch.empty_like(x), torch.empty_like(x)
    call(x, before, out, want, layer.workspace(B, L))
    rest = buf.clone()
    call(x, buf[:n] if shift > 16 else before, out2, buf[shift:shift + n], layer.workspace(B, L))
    assert torch.equal(out, out2) and torch.equal(buf[shift:shift + n], want)
    assert torch.equal(buf[:shift], rest[:shift]) and torch.equal(buf[shift + n:], rest[shift + n:])
