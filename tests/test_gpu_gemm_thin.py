"""The routed GEMM with a narrow fp32 output (x projection; backward of the dt projection): rows at the edges of its 32-row blocks
and of its rule, one to five blocks of columns, whole and ragged, fewer slabs than its ring and slices of the contraction, uneven and
empty groups; B and C against products in 64 bits (an fp32 sum of K terms: 2^-24 of the terms' size for each addition that it can
have been rounded in, at most K / 16 + 24), the backward against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import TOL, rel_err, to_np

pytestmark = pytest.mark.gpu


def cfg_of(n, rank, d_inner, E, K=1, bias=None):
    return RomConfig(f"thin_{n}_{rank}", 930 + rank % 31, 1, n, 64, d_inner, 16, 4, rank, E, K, "bf16", int(K > 1), router_bias=bias)


@pytest.mark.parametrize("n,rank,d_inner,E,K,bias", [
    (1023, 16, 256, 1, 1, None), (1024, 16, 64, 1, 1, None), (1025, 8, 128, 3, 1, None), (1057, 32, 192, 4, 1, (9.0, 0.0, 0.0, -50.0)),
    (1300, 40, 1088, 8, 1, None), (3001, 64, 512, 8, 1, None), (2500, 72, 1024, 5, 1, (9.0, 0.0, 0.0, 0.0, -50.0)),
    (1100, 96, 2048, 16, 2, None), (2047, 104, 320, 2, 2, None), (5000, 128, 1024, 8, 1, None), (1024, 128, 4096, 64, 1, None),
    (40000, 64, 256, 6, 1, None), (20000, 128, 192, 3, 1, (9.0, 0.0, -50.0)), (33000, 24, 128, 2, 2, None),
    (500, 48, 1024, 64, 1, None),                               # few rows, but many groups
])
def test_thin_forward(n, rank, d_inner, E, K, bias):
    cfg = cfg_of(n, rank, d_inner, E, K, bias)
    layer = RomLayer(cfg, make_weights(cfg))
    layer.forward(layer.to_device(make_input(cfg)))
    u, idx, w = layer.ws_view("u", 1, n).double(), layer.ws_view("expert_idx", 1, n), layer.weights["w_x"].double()
    ref = torch.zeros(n, rank + 32, dtype=torch.float64, device=u.device)
    size = torch.zeros_like(ref)
    for k in range(K):
        for e in range(E):
            rows = (idx[:, k] == e).nonzero().flatten()
            ref[rows] += u[rows] @ w[e].T
            size[rows] += u[rows].abs() @ w[e].T.abs()
    tol = 2.0 ** -24 * (d_inner / 16 + 24)
    assert ((layer.ws_view("bc", 1, n).double() - ref[:, rank:]).abs() <= tol * size[:, rank:]).all()
    low = layer.ws_view("dt_low", 1, n).double()
    assert ((low - ref[:, :rank]).abs() <= 2.0 ** -8 * ref[:, :rank].abs() + 1.01 * tol * size[:, :rank]).all()


@pytest.mark.parametrize("n,rank,d_inner,E,K", [(1100, 32, 320, 3, 1), (1030, 128, 256, 2, 1), (1200, 72, 512, 4, 2)])
def test_thin_backward(n, rank, d_inner, E, K):
    cfg = cfg_of(n, rank, d_inner, E, K)
    w, x = make_weights(cfg), make_input(cfg)
    layer = RomLayer(cfg, w)
    layer.forward(layer.to_device(x))
    idx = to_np(layer.ws_view("expert_idx", 1, n))
    d_out = layer.to_device(np.random.default_rng(n).standard_normal((1, n, 64)).astype(np.float32))
    d_x, grads = layer.backward(layer.to_device(x), d_out)
    torch.cuda.synchronize()
    ref = O.rom_layer_backward(x, w, cfg.top_k, cfg.gate_mode, to_np(d_out), expert_idx=idx)
    assert rel_err(to_np(d_x), ref["d_x"]) <= TOL["bf16"]
    for name in ("d_w_in", "d_w_x", "d_w_dt", "d_A_log"):
        assert rel_err(to_np(grads[name]), ref[name]) <= TOL["bf16"], name
