"""The row kernels at the edges of their layout: 2^k lanes per token for K entries, segments of 64 tokens, batches held in
registers once (T 2^k <= 8192) or read again, one block up to 1024 tokens and one segment per block beyond."""
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._util import check_route, oracle_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,m,K,way,Ns,full", [
    (1, 8, 1, 2, 0, False), (1, 256, 32, 8, 8, False), (63, 20, 3, 4, 1, False), (65, 256, 32, 1, 2, False),
    (256, 64, 32, 64, 0, False), (257, 64, 32, 5, 1, True), (1024, 128, 8, 8, 0, False), (1023, 96, 17, 8, 1, False),
    (1024, 40, 9, 256, 8, False), (1025, 256, 32, 8, 1, False), (1088, 5, 5, 2, 0, False), (1089, 250, 8, 3, 2, True)])
@pytest.mark.parametrize("threshold", [0.0, 0.45, 1.0])
def test_rows_at_the_edges_of_the_layout(T, m, K, way, Ns, full, threshold):
    print(T, m, K, way, Ns, full, threshold, flush=True)
    cfg = WL.LayerConfig("rows", T=T, d=64, F=64, m=m, K=K, way=way, n_shared=Ns, F_s=64 if Ns else 0, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    x, gate_w = L.x.to("cuda"), L.gate_w.to("cuda")
    gate_b = None if L.gate_b is None else L.gate_b.to("cuda")
    R = P.moe_route(P.config_of(cfg), x, gate_w, gate_b, threshold, full)
    torch.cuda.synchronize()
    check_route(R, oracle_route(L, cfg, threshold, full), cfg, threshold, full)
