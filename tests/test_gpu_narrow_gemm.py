"""The narrow GEMM (few blocks of small tiles): one k tile and fewer than its stages, both tile heights with full and ragged
tiles, one, two and four K slices, shared experts in a launch of their own; and a batch of 128-row tiles next to it."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._util import OUT_TOL, check_route, npf, oracle_route, rel_err

pytestmark = pytest.mark.gpu


# T, d, F, m, K, way, n_shared, F_s
@pytest.mark.parametrize("T,d,F,m,K,way,Ns,Fs", [
    (1, 64, 64, 1, 1, 2, 0, 0), (1, 1024, 192, 128, 8, 8, 2, 192), (31, 320, 448, 3, 1, 2, 1, 64), (33, 64, 2048, 2, 2, 2, 0, 0),
    (37, 384, 128, 60, 4, 8, 1, 1408), (64, 448, 1024, 2, 1, 2, 0, 0), (65, 192, 64, 8, 2, 8, 1, 960), (128, 256, 128, 8, 2, 4, 2, 320),
    (129, 256, 128, 8, 2, 4, 1, 320), (40, 128, 128, 4, 1, 4, 0, 0), (96, 64, 128, 64, 8, 8, 0, 0), (640, 128, 192, 64, 8, 8, 0, 0)])
@pytest.mark.parametrize("threshold", [1.0, 0.5])
def test_small_tiles(T, d, F, m, K, way, Ns, Fs, threshold):
    print(T, d, F, m, K, way, Ns, Fs, threshold, flush=True)
    cfg = WL.LayerConfig("narrow", T=T, d=d, F=F, m=m, K=K, way=way, n_shared=Ns, F_s=Fs, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    to = lambda t: None if t is None else t.to("cuda")
    x, gate_w, gate_b = to(L.x), to(L.gate_w), to(L.gate_b)
    experts = tuple(to(a) for a in L.experts)
    shared = None if L.shared is None else tuple(to(a) for a in L.shared)
    united_cpu = WL.make_random_united(cfg, 1, "cpu")
    united = tuple(to(a) for a in united_cpu)
    c = P.config_of(cfg)
    ws = P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    R = P.moe_route(c, x, gate_w, gate_b, threshold, False, workspace=ws)
    torch.cuda.synchronize()
    idx, w, unit = check_route(R, oracle_route(L, cfg, threshold, False), cfg, threshold, False)
    got = npf(P.moe_forward(c, x, gate_w, gate_b, experts, united, shared, threshold, False, workspace=ws))
    want = O.forward_tokens(npf(L.x), idx, w, unit, way, npf(L.experts), npf(united_cpu), npf(L.shared))
    assert np.isfinite(got).all()
    assert rel_err(got, want) <= OUT_TOL


# m, K, d, F and batch sizes whose experts' rows go through different kernels: narrow with 32 and 64 rows and the 128-row
# kernel for few experts (28 to 56 blocks of 256 columns), narrow with 32 rows and the 64-row kernel for 64 experts.  F < 1024:
# one K slice; the gate sums in one order at all of these sizes.
@pytest.mark.parametrize("m,K,d,F,sizes", [(8, 2, 1024, 896, (20, 100, 600)), (64, 8, 128, 960, (3, 96))])
def test_the_kernel_of_a_launch_does_not_show_in_the_bits(m, K, d, F, sizes):
    print(m, K, d, F, sizes, flush=True)
    cfg = WL.LayerConfig("narrow_bits", T=max(sizes), d=d, F=F, m=m, K=K, way=8)
    L = WL.make_layer(cfg, 5, "cpu")
    x, gate_w, gate_b = L.x.to("cuda"), L.gate_w.to("cuda"), None if L.gate_b is None else L.gate_b.to("cuda")
    experts = tuple(a.to("cuda") for a in L.experts)
    c = P.config_of(cfg)
    out = {T: P.moe_forward(c, x[:T].contiguous(), gate_w, gate_b, experts) for T in sizes}
    torch.cuda.synchronize()
    for T in sizes[1:]:
        assert torch.equal(out[T][:sizes[0]], out[sizes[0]]), T
