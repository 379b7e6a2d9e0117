"""A backward workspace of the largest call serves the smaller ones where the conv adjoint's runs and the router's chunks get
shorter (host planning; the adjoint scan's chunks are 128 steps at all of these sizes)."""
import pytest

from paper_2506_18145_amd.binding import RomDims, rom_backward_workspace_bytes


@pytest.mark.parametrize("d_inner,calls", [
    (2048, [(b, 128) for b in range(240, 262)]), (2048, [(1, n) for n in range(8150, 8230)]),
    (4096, [(1, n) for n in range(16250, 16390, 3)]), (2048, [(b, 1) for b in range(4085, 4105)]),
    (1600, [(64, n) for n in range(120, 520, 7)]),
])
def test_smaller_calls_need_no_more(d_inner, calls):
    dims = RomDims(d_model=d_inner // 2, d_inner=d_inner, d_state=16, d_conv=4, dt_rank=64, n_experts=8, top_k=1, n_experts_xdt=8,
                   dtype=1, gate_mode=0)
    sizes = [rom_backward_workspace_bytes(dims, b, n) for b, n in calls]
    assert sizes[0] > 0 and sizes == sorted(sizes)
