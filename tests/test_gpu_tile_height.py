"""Tile heights of batches with many experts, whose fuller units want more rows than the mean: the kernels on both sides of each
step (3 and 4 rows per expert, 11 and 12), next to shared experts of a width of their own (256 and 257 tokens), and the height of
those (256 rows from a tile for every CU on)."""
import re

import numpy as np
import pytest

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._fake_hip import trace
from tests._util import OUT_TOL, npf, oracle_route, rel_err

# T, n_shared, F_s, kernel of GEMM1 (routed, then shared experts of another width)
M, K, D, F = 20, 2, 1024, 1664
CASES = [(30, 0, 0, ["32"]), (40, 0, 0, ["64"]), (119, 0, 0, ["64"]), (120, 0, 0, ["ws"]), (120, 1, F, ["ws"]),
         (256, 1, 192, ["pair 64"]), (257, 1, 192, ["ws", "ws"]), (600, 1, 10880, ["ws", "ws"]), (600, 1, 10944, ["ws", "w4"])]


def _kernels(launches):
    names = {"ffn_gemm_ws_kernel": "ws", "ffn_gemm_w4_kernel": "w4"}
    found = []
    for l in launches:
        if not l["name"].startswith("ffn_gemm") or "Lb1EEEvNS" not in l["symbol"]:       # GEMM1: <..., true>
            continue
        height = re.search(r"ILi(\d+)E", l["symbol"])
        found.append(names.get(l["name"]) or ("pair " if "pair" in l["name"] else "") + height.group(1))
    return found


def test_kernels_of_the_cases(tmp_path):
    calls = [dict(entry="forward", cfg=[D, F, M, K, 4, ns, fs, 0, 0, 0], T=T, threshold=1.0) for T, ns, fs, _ in CASES]
    for c, r in zip(CASES, trace(calls, tmp_path)):
        assert r["status"] == 0 and _kernels(r["launches"]) == c[3], (c, _kernels(r["launches"]))


@pytest.mark.gpu
@pytest.mark.parametrize("T,ns,fs", [c[:3] for c in CASES])
@pytest.mark.parametrize("threshold", [1.0, 0.5])
def test_against_the_oracle(T, ns, fs, threshold):
    print(T, ns, fs, threshold, flush=True)
    cfg = WL.LayerConfig("height", T=T, d=D, F=F, m=M, K=K, way=4, n_shared=ns, F_s=fs, zipf_s=1.0)
    L = WL.make_layer(cfg, T + ns, "cpu")
    to = lambda t: None if t is None else tuple(a.to("cuda") for a in t)
    united_cpu = WL.make_random_united(cfg, 1, "cpu")
    c = P.config_of(cfg)
    ws = P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    got = npf(P.moe_forward(c, L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda"), to(L.experts), to(united_cpu), to(L.shared),
                            threshold, False, workspace=ws))
    r = oracle_route(L, cfg, threshold)
    tokens = np.nonzero(r.margin >= 1e-6)[0]
    tokens = tokens[np.unique(np.linspace(0, len(tokens) - 1, 48).astype(int))].astype(np.int32)
    want = O.forward_tokens(npf(L.x), r.topk_idx, r.topk_w, r.expert_unit, 4, npf(L.experts), npf(united_cpu), npf(L.shared), tokens=tokens)
    assert np.isfinite(got).all()
    assert rel_err(got[tokens], want) <= OUT_TOL
