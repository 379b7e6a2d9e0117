"""A sequence's results do not depend on the other sequences of its call: in two calls of the same shape it has the same bits, forward
and backward, wherever the others' tokens push its rows in the grouping."""
import numpy as np
import pytest
import torch

from paper_2506_18145_amd import RomLayer
from rom_synth import RomConfig, make_input, make_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,d_model,d_inner,rank,E,K,dtype", [
    (700, 256, 1024, 16, 8, 1, "bf16"), (401, 128, 2048, 96, 8, 1, "bf16"), (600, 128, 512, 64, 16, 2, "bf16"),
    (3000, 64, 768, 32, 5, 1, "bf16"), (450, 64, 512, 32, 4, 1, "fp32"),
])
def test_same_bits_in_other_company(L, d_model, d_inner, rank, E, K, dtype):
    cfg = RomConfig(f"mates_{L}", 940 + L % 31, 3, L, d_model, d_inner, 16, 4, rank, E, K, dtype, int(K > 1))
    layer = RomLayer(cfg, make_weights(cfg))
    x = layer.to_device(make_input(cfg))
    d_out = layer.to_device(np.random.default_rng(L).standard_normal((3, L, d_model)).astype(np.float32))
    other = torch.cat([x[:1], x[1:].flip(1, 2) * 0.5])
    got = []
    for xi in (x.contiguous(), other.contiguous()):
        out, conv, ssm = layer.forward(xi, return_states=True)
        bc = layer.ws_view("bc", 3, L).view(3, L, -1)[0].clone()
        low = layer.ws_view("dt_low", 3, L).view(3, L, -1)[0].clone()
        d_x, _ = layer.backward(xi, d_out)
        torch.cuda.synchronize()
        got.append((bc, low, out[0].clone(), conv[0].clone(), ssm[0].clone(), d_x[0].clone()))
    for a, b in zip(*got):
        assert torch.equal(a, b)
