"""The 128-row GEMM (waves that load, waves that multiply): one k tile and fewer than its stages, column tiles of either width, full
and ragged row tiles, several tiles per block, K slices and shared experts narrower than those (slices without any k)."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._util import OUT_TOL, npf, oracle_route, rel_err

pytestmark = pytest.mark.gpu


# T, d, F, m, K, way, n_shared, F_s: 48 to 383 rows per expert
@pytest.mark.parametrize("T,d,F,m,K,way,Ns,Fs", [
    (48, 64, 64, 1, 1, 1, 0, 0), (127, 128, 192, 1, 1, 1, 0, 0), (129, 64, 8192, 1, 1, 1, 0, 0), (129, 64, 16448, 1, 1, 1, 0, 0),
    (300, 64, 16384, 2, 2, 2, 0, 0), (256, 4160, 576, 2, 1, 2, 0, 0), (383, 320, 4096, 4, 2, 2, 1, 64), (383, 448, 1088, 3, 3, 3, 1, 1088),
    (1500, 192, 704, 12, 1, 4, 2, 704)])
@pytest.mark.parametrize("threshold", [1.0, 0.5])
def test_against_the_oracle(T, d, F, m, K, way, Ns, Fs, threshold):
    print(T, d, F, m, K, way, Ns, Fs, threshold, flush=True)
    cfg = WL.LayerConfig("streaming", T=T, d=d, F=F, m=m, K=K, way=way, n_shared=Ns, F_s=Fs, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    to = lambda t: None if t is None else t.to("cuda")
    experts = tuple(to(a) for a in L.experts)
    shared = None if L.shared is None else tuple(to(a) for a in L.shared)
    united_cpu = WL.make_random_united(cfg, 1, "cpu")
    united = tuple(to(a) for a in united_cpu)
    c = P.config_of(cfg)
    ws = P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    got = npf(P.moe_forward(c, to(L.x), to(L.gate_w), to(L.gate_b), experts, united, shared, threshold, False, workspace=ws))
    r = oracle_route(L, cfg, threshold)
    tokens = np.nonzero(r.margin >= 1e-6)[0]
    tokens = tokens[np.unique(np.linspace(0, len(tokens) - 1, 96).astype(int))].astype(np.int32)
    want = O.forward_tokens(npf(L.x), r.topk_idx, r.topk_w, r.expert_unit, way, npf(L.experts), npf(united_cpu), npf(L.shared), tokens=tokens)
    assert np.isfinite(got).all()
    assert rel_err(got[tokens], want) <= OUT_TOL
