"""SwiGLU of the trainer in 256 x 192 tiles (several groups side by side) and in 128 x 128 ones (one group at a time): the same bits, with
ragged last tiles in both directions."""
import ctypes as C

import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL

pytestmark = pytest.mark.gpu


# four groups: 576 small tiles (a round of two blocks on a CU and one of one) or 220 large ones (one round); one k tile and several
@pytest.mark.parametrize("d", [64, 320])
@pytest.mark.parametrize("n", [1088, 1152])
def test_same_bits(n, d):
    cfg = WL.LayerConfig("tiles", T=n, d=d, F=1024, m=8, K=2, way=2)
    L = WL.make_layer(cfg, 1, "cpu")
    experts = tuple(a.to("cuda") for a in L.experts)
    x = WL.make_activations(cfg, 1, "cpu", "calib", n).to("cuda")
    c = P.config_of(cfg)
    wanted = C.c_size_t(0)
    assert P.lib().moe_distill_workspace_size(C.byref(c), n, C.byref(wanted)) == 0

    def train(size):
        united = tuple(u.to("cuda") for u in WL.make_random_united(cfg, 2, "cpu"))
        ws = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        return united + (P.moe_distill_united(c, experts, united, x, 2, 1e-3, workspace=ws),)

    side = train(wanted.value)
    one = (wanted.value - P.workspace_size(c, n)) // 4 + P.workspace_size(c, n) + (1 << 20)     # one group and part of another
    for a, b in zip(side, train(one)):
        assert torch.equal(a, b)
    assert torch.isfinite(side[3]).all() and (side[3][:, 1:] < side[3][:, :1]).all()
