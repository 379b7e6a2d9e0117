"""Grouping and router at the lines of their rules: the edges of a workgroup's rounds and of one workgroup against three
launches (stable order, exact), and four wavefronts or one for a token (logits and gates against the oracle, the logits of up to
8192 tokens against 64 bits; the router of a block reads the normalised input)."""
import numpy as np
import pytest
import torch

from oracle import rom_oracle as O
from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights
from gpu_util import BLOCK_EPS, check_routing, to_np

pytestmark = pytest.mark.gpu


def layer_of(n, d_model, E, K, dtype="bf16", bias=None):
    cfg = RomConfig(f"route_{n}", 900 + n % 89, 1, n, d_model, 64, 16, 4, 8, E, K, dtype, K > 1, router_bias=bias)
    w = make_weights(cfg)
    return cfg, w, RomLayer(cfg, w)


@pytest.mark.parametrize("E,K,tokens", [
    (8, 1, (1, 64, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193)),
    (16, 1, (257, 2049, 4096, 4097)), (17, 1, (1025, 2048, 2049)), (64, 1, (257, 1024, 2048, 2049)),
    (1, 1, (1000, 8192)), (5, 3, (86, 342, 683, 2730, 2731)), (64, 8, (33, 128, 256, 257)),
])
@pytest.mark.parametrize("skewed", [False, True])
def test_grouping_edges(E, K, tokens, skewed):
    bias = None if not skewed else tuple(9.0 if e == E - 1 else -9.0 if e == 0 and E > K else 0.0 for e in range(E))
    _, _, layer = layer_of(max(tokens), 64, E, K, bias=bias)
    x = layer.to_device(np.random.default_rng(E).standard_normal((max(tokens), 64)).astype(np.float32))
    for n in tokens:
        r = {k: to_np(v) for k, v in layer.route(x[:n]).items()}
        want = O.expert_permutation(r["expert_idx"], E)
        for name, ref in zip(("counts", "offsets", "perm", "inv_perm"), want):
            assert np.array_equal(r[name], ref), (n, name)


@pytest.mark.parametrize("n,d_model,E,K,dtype", [
    (1024, 512, 8, 1, "bf16"), (1025, 512, 8, 1, "bf16"), (3072, 544, 8, 1, "bf16"), (3073, 544, 8, 2, "bf16"),
    (4096, 1024, 8, 1, "bf16"), (4097, 1024, 5, 1, "bf16"), (4097, 1032, 8, 1, "bf16"), (4097, 1024, 8, 1, "fp32"),
    (3072, 768, 16, 2, "bf16"), (3073, 768, 16, 1, "bf16"), (3073, 776, 12, 1, "bf16"), (3072, 1024, 16, 1, "fp32"),
])
@pytest.mark.parametrize("block", [False, True])
def test_router_rule(n, d_model, E, K, dtype, block):
    cfg, w, layer = layer_of(n, d_model, E, K, dtype)
    x_np = make_input(cfg)
    x = layer.to_device(x_np)
    if block:
        layer.block_forward(x, eps=BLOCK_EPS)
    else:
        layer.forward(x)
    torch.cuda.synchronize()
    names = ("expert_idx", "gate", "counts", "offsets", "perm", "inv_perm", "logits")
    check_routing(cfg, {k: to_np(layer.ws_view(k, 1, n)) for k in names}, x_np, w, block)


@pytest.mark.parametrize("n,d_model,E", [(8192, 1024, 8), (5000, 2048, 8), (4097, 768, 5), (6000, 1536, 16), (3073, 768, 16)])
@pytest.mark.parametrize("block", [False, True])
def test_router_precision(n, d_model, E, block):
    """Up to 8192 tokens a logit is at most d_model / 64 additions in a lane and six over the lanes.  An addition is off by up to
    2^-24 of what it leaves, evenly spread (2^-24 / sqrt(3) rms), so the logits by that times the root of (d_model / 64 + 1) / 2 + 6 (sums
    of part of the terms are smaller by the root of their part); a block adds two roundings a term and some four of 1 / rms."""
    cfg, w, layer = layer_of(n, d_model, E, 1)
    x_np = make_input(cfg)
    x = layer.to_device(x_np)
    layer.block_forward(x, eps=BLOCK_EPS) if block else layer.forward(x)
    torch.cuda.synchronize()
    x_r = (O.rms_norm(x_np, w["norm_w"], BLOCK_EPS) if block else x_np).reshape(n, -1)
    ref = O.router_logits(x_r, w["w_router"], w.get("b_router"))
    err = np.linalg.norm(to_np(layer.ws_view("logits", 1, n)).astype(np.float64) - ref) / np.linalg.norm(ref)
    assert err <= 2.0 ** -24 / 3 ** 0.5 * ((d_model / 64 + 1) / 2 + 6 + (6 if block else 0)) ** 0.5
