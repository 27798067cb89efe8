"""Routing where the choice of its kernels changes: TopK inside the routing block (up to 64 tokens; a few by rank) or before it, bitmaps from the
TopK launch or from the lists, one launch for the rows or three, logits that do not fit the scratch in one piece."""
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._util import check_route, npf, oracle_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,m,K,way,Ns,d", [
    (64, 16, 16, 3, 1, 64), (64, 16, 15, 8, 0, 64), (64, 17, 16, 4, 0, 64), (64, 256, 15, 8, 2, 64), (33, 200, 20, 7, 1, 1024),
    (5, 130, 8, 8, 0, 2048),                                                    # one block, 8 slices of K
    (1, 128, 8, 8, 0, 2048), (2, 120, 15, 8, 0, 64), (3, 128, 8, 8, 0, 64), (4, 60, 4, 8, 1, 2048), (5, 64, 4, 8, 0, 64),
    (1, 256, 8, 8, 1, 1024), (8, 17, 8, 2, 0, 64),                              # winners by rank, and just too many tokens for it
    (12, 256, 1, 8, 0, 1024), (31, 256, 1, 8, 0, 1024),                         # pieces of 8 (lists) and of 16 tokens (bits)
    (65, 17, 2, 2, 0, 64), (127, 64, 1, 64, 0, 64), (2049, 16, 2, 8, 1, 64),    # lists of few experts, both gates
    (8192, 128, 2, 8, 0, 64), (8193, 40, 2, 8, 1, 64),                          # 128 segments and one more
    (4096, 256, 2, 1, 0, 64), (4160, 256, 2, 16, 0, 64), (4224, 256, 2, 5, 0, 64)])    # bitmaps that fit the LDS, and that do not
@pytest.mark.parametrize("threshold,full", [(1.0, False), (0.4, False), (0.0, True)])
def test_against_the_oracle(T, m, K, way, Ns, d, threshold, full):
    print(T, m, K, way, Ns, d, threshold, full, flush=True)
    cfg = WL.LayerConfig("rows", T=T, d=d, F=64, m=m, K=K, way=way, n_shared=Ns, F_s=64 if Ns else 0, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    R = P.moe_route(P.config_of(cfg), L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda"), threshold, full)
    torch.cuda.synchronize()
    check_route(R, oracle_route(L, cfg, threshold, full), cfg, threshold, full)


@pytest.mark.parametrize("m,K", [(8, 3), (16, 16), (5, 5)])
def test_few_experts_some_of_logit_minus_infinity(m, K):
    """A masked expert is picked once, after the others and with weight 0, in the routing block (64 tokens) as in the gate's own
    TopK (65)."""
    print(m, K, flush=True)
    cfg = WL.LayerConfig("mask", T=65, d=128, F=64, m=m, K=K, way=2)
    L = WL.make_layer(cfg, m, "cpu")
    x, gw = L.x.to("cuda"), L.gate_w.to("cuda")
    bias = torch.zeros(m)
    bias[[e for e in range(m) if e % 3 == 1 or e > K // 2]] = float("-inf")
    c = P.config_of(cfg)
    big = P.moe_route(c, x, gw, bias.to("cuda"), 0.5)
    small = P.moe_route(c, x[:64].contiguous(), gw, bias.to("cuda"), 0.5)
    torch.cuda.synchronize()
    assert all(len(set(r)) == K for r in npf(small.topk_idx).tolist())
    for f in ("topk_idx", "topk_w", "near_tie"):
        assert torch.equal(getattr(big, f)[:64], getattr(small, f)), f
