"""A token's output has the same bits whichever GEMM kernel its batch gets: 32-, 64- and 128-row tiles, a quarter of the columns per block, 128-
or 256-column tiles of the streaming kernel, routed units and shared experts in one launch or two.  One plane of GEMM2 in all (F below
1024) and no 256-row tiles, whose tail may be cut along K."""
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._fake_hip import trace

MOST = 1000
SIZES = [7, 20, 100, 220, 256, 300, 700]
# d, F, n_shared, F_s (40 experts, top 2)
SHAPES = [(1024, 960, 0, 0), (1024, 960, 1, 192), (1152, 960, 2, 960), (512, 320, 0, 0), (512, 320, 1, 1600)]
KERNELS = {"ffn_gemm_kernel", "ffn_gemm_narrow_kernel", "ffn_gemm_either_kernel", "ffn_gemm_pair_kernel", "ffn_gemm_ws_kernel"}


def test_the_sizes_take_all_kernels(tmp_path):
    calls = [dict(entry="forward", cfg=[d, F, 40, 2, 8, ns, fs, 0, 0, 0], T=T, own_route=1, threshold=1.0)
             for d, F, ns, fs in SHAPES for T in SIZES + [MOST]]
    got = trace(calls, tmp_path)
    assert all(r["status"] == 0 and r["launches"][-1]["planes"] == 1 for r in got)
    names = [{l["name"] for l in r["launches"] if l["name"].startswith("ffn_gemm")} for r in got]
    assert set().union(*names) == KERNELS
    assert all(n == {"ffn_gemm_ws_kernel"} for c, n in zip(calls, names) if c["T"] == MOST and c["cfg"][6] < 1024)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("zipf", [None, 1.0])
def test_same_bits(shape, zipf):
    d, F, ns, fs = shape
    print(shape, zipf, flush=True)
    cfg = WL.LayerConfig("bits", T=MOST, d=d, F=F, m=40, K=2, way=8, n_shared=ns, F_s=fs, zipf_s=zipf)
    L = WL.make_layer(cfg, d + F, "cuda")
    c = P.config_of(cfg)

    def forward(T, weights=None):
        x = L.x[:T].contiguous()
        R = P.moe_route(c, x, L.gate_w, L.gate_b, 1.0)
        if weights is not None:                   # the gate may cut K otherwise in another batch: the same row weights
            R.row_weight[R.token_rows[:, :2].long()] = weights[:T]
        return R, P.moe_forward(c, x, L.gate_w, L.gate_b, L.experts, None, L.shared, route=R)

    R, want = forward(MOST)
    for T in SIZES:
        r, got = forward(T, R.topk_w)
        assert torch.equal(r.topk_idx, R.topk_idx[:T])
        assert torch.equal(got, want[:T]), T
