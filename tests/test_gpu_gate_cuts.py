"""The many-expert gate at the places where it is cut: blocks of 16, 64 and 128 tokens and of 64 experts, slices of K,
TopK of 16 lanes or a wavefront per token, and batches that go through its scratch in pieces (moe_route_static)."""
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._util import check_route, oracle_route

pytestmark = pytest.mark.gpu


# T, d, m, K: one token; edges of 16 and 64 tokens and of 64 experts; one k step (no slices), a prime number of them;
# K + 1 = 16 picks and more; the last size of 16-token blocks and the next; the first of 128-token blocks and the one before
@pytest.mark.parametrize("T,d,m,K", [
    (1, 64, 17, 1), (1, 2048, 128, 8), (15, 192, 64, 15), (17, 832, 65, 16), (63, 448, 129, 8), (64, 128, 33, 32),
    (65, 1024, 250, 8), (512, 576, 256, 8), (513, 576, 256, 8), (2049, 704, 60, 4), (8191, 64, 256, 3), (8192, 128, 256, 8),
    (8193, 64, 200, 31)])
def test_routing_at_the_cuts_of_the_gate(T, d, m, K):
    print(T, d, m, K, flush=True)
    cfg = WL.LayerConfig("gate_cut", T=T, d=d, F=64, m=m, K=K, way=8, zipf_s=1.0, score_fn=T % 2)
    L = WL.make_layer(cfg, T + m, "cpu")
    x, gate_w, gate_b = L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda")
    c = P.config_of(cfg)
    R = P.moe_route(c, x, gate_w, gate_b, 0.5)
    torch.cuda.synchronize()
    check_route(R, oracle_route(L, cfg, 0.5), cfg, 0.5, False)


# d = 128: K is not sliced; the rest: two to eight slices, which the pieces of the smaller scratch have to keep
@pytest.mark.parametrize("T,d,m", [(2048, 128, 256), (2049, 128, 256), (9000, 128, 256), (2048, 7168, 256), (8192, 2048, 128),
                                   (300, 1088, 200), (1021, 4096, 256), (40, 1024, 17), (4999, 2048, 60)])
def test_a_batch_in_pieces_routes_like_the_whole(T, d, m):
    print(T, d, m, flush=True)
    cfg = WL.LayerConfig("gate_pieces", T=T, d=d, F=1024, m=m, K=4, way=8, zipf_s=1.0)
    L = WL.make_layer(cfg.with_(F=64), T, "cuda")
    c = P.config_of(cfg)
    L.gate_w, c = P.pack_gate(c, L.gate_w), P.with_packed_gate(c)
    want = P.moe_route(c, L.x, L.gate_w, L.gate_b, 0.4)
    got = P.alloc_route_out(c, T)
    P.moe_route_static(c, L.x, L.gate_w, L.gate_b, 0.4, False, got)
    torch.cuda.synchronize()
    n = int(want.n_rows.item())
    for f in ("topk_idx", "topk_w", "expert_cnt", "expert_unit", "unit_cnt", "unit_off", "token_rows", "n_rows", "near_tie"):
        assert torch.equal(getattr(got, f), getattr(want, f)), f
    assert torch.equal(got.row_token[:n], want.row_token[:n])
    assert torch.equal(got.row_weight[:n], want.row_weight[:n])
