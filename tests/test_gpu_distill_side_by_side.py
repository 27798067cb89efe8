"""Groups trained side by side and one at a time: the same weights and losses bit for bit, whatever the workspace holds."""
import ctypes as C

import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import binding as B
from paper_2507_17133_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _bytes(c, n):
    b = C.c_size_t(0)
    assert P.lib().moe_distill_workspace_size(C.byref(c), n, C.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("n", [64, 448])
def test_same_results(n):
    cfg = WL.LayerConfig("side_by_side", T=n, d=192, F=448, m=11, K=2, way=2)      # five pairs and a lone member
    L = WL.make_layer(cfg, 1, "cpu")
    experts = tuple(a.to("cuda") for a in L.experts)
    x = WL.make_activations(cfg, 1, "cpu", "calib", n).to("cuda")
    c = P.config_of(cfg)
    def train(size):
        united = tuple(u.to("cuda") for u in WL.make_random_united(cfg, 2, "cpu"))
        ws = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        return united + (P.moe_distill_united(c, experts, united, x, 3, 1e-3, workspace=ws),)

    got, one = [], P.workspace_size(c, n)
    while not got:                                     # the least it takes, to 256 KiB: room for one group
        one += 1 << 18
        try:
            got.append(train(one))
        except P.MoeError as e:
            assert e.status == -4 and one < _bytes(c, n)
    assert one + 38 * 192 * 448 < _bytes(c, n)         # two do not fit in it
    got += [train(_bytes(c, n)), train(_bytes(c, 4096))]
    torch.cuda.synchronize()
    for g in got[1:]:
        for a, b in zip(got[0], g):
            assert torch.equal(a, b)
