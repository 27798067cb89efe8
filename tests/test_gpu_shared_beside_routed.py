"""Shared experts of a width of their own in decode-sized batches, whose GEMMs go out together with the routed units': each pair of
tile heights and kernels (1 to 12 tokens: 32-row tiles of both; more: 64-row tiles of the shared experts), K slices, brownout, and
batches just beyond."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._fake_hip import trace
from tests._util import OUT_TOL, npf, oracle_route, rel_err

# T, d, F, m, K, way, n_shared, F_s and the pair of the two GEMMs' kernels (rows of the routed tiles, narrow, of the shared ones)
CASES = [(1, 128, 64, 8, 2, 4, 1, 192, "32,1,32", "32,1,32"), (20, 512, 1024, 64, 8, 8, 1, 2048, "32,0,32", "32,0,32"),
         (37, 256, 1088, 60, 4, 8, 1, 2112, "32,0,64", "32,1,64"), (64, 128, 192, 4, 1, 2, 2, 320, "32,1,64", "32,1,64"),
         (100, 192, 2112, 64, 8, 8, 1, 1088, "64,0,64", "64,0,64"),
         (100, 256, 1408, 24, 4, 8, 1, 1088, "64,0,64", "64,1,64"), (128, 640, 128, 24, 4, 8, 1, 64, "32,1,64", "32,1,64"),
         (256, 256, 128, 24, 4, 8, 1, 320, "64,1,64", "64,1,64"),
         (257, 256, 128, 24, 4, 8, 1, 320, None, None), (383, 64, 128, 24, 4, 8, 1, 320, None, None)]


def _pairs(launches):
    import re
    found = []
    for l in launches:
        if l["name"] == "ffn_gemm_pair_kernel":
            r, n, s = re.search(r"ILi(\d+)ELb(\d)ELi(\d+)E", l["symbol"]).groups()
            found.append(f"{r},{n},{s}")
    return found or [None, None]


def test_kernels_of_the_cases(tmp_path):
    calls = [dict(entry="forward", cfg=[d, F, m, K, way, Ns, Fs, 0, 0, 0], T=T, threshold=1.0)
             for T, d, F, m, K, way, Ns, Fs, _, _ in CASES]
    for c, r in zip(CASES, trace(calls, tmp_path)):
        assert r["status"] == 0 and _pairs(r["launches"]) == list(c[8:]), (c, _pairs(r["launches"]))


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("threshold", [1.0, 0.5])
def test_against_the_oracle(case, threshold):
    T, d, F, m, K, way, Ns, Fs = case[:8]
    print(case, threshold, flush=True)
    cfg = WL.LayerConfig("beside", T=T, d=d, F=F, m=m, K=K, way=way, n_shared=Ns, F_s=Fs, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    to = lambda t: tuple(a.to("cuda") for a in t)
    united_cpu = WL.make_random_united(cfg, 1, "cpu")
    c = P.config_of(cfg)
    ws = P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    got = npf(P.moe_forward(c, L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda"), to(L.experts), to(united_cpu), to(L.shared),
                            threshold, False, workspace=ws))
    r = oracle_route(L, cfg, threshold)
    tokens = np.nonzero(r.margin >= 1e-6)[0].astype(np.int32)
    want = O.forward_tokens(npf(L.x), r.topk_idx, r.topk_w, r.expert_unit, way, npf(L.experts), npf(united_cpu), npf(L.shared), tokens=tokens)
    assert np.isfinite(got).all()
    assert rel_err(got[tokens], want) <= OUT_TOL
