"""Left-over 256-row tiles of the shared experts, whose number the host knows: cut along K, with the sum of the slices behind the GEMM, or
not, and then without it."""
import numpy as np
import pytest

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._fake_hip import trace
from tests._util import OUT_TOL, npf, oracle_route, rel_err

# T, d, F_s; sums behind GEMM1 and GEMM2 of the shared expert (256 CUs).  4 tiles left over of 260 and 20 on 56 blocks; K 256 too short, and 2
# tiles of K 16384; whole rounds, and 8 tiles on 24 blocks; 5 tiles left over of 261, and 144 on 256 blocks
CASES = [(1025, 1024, 6656, 1, 1), (400, 256, 16384, 0, 1), (400, 1024, 16384, 0, 1), (2049, 4096, 3712, 1, 0)]


def _cfg(T, d, Fs):
    return WL.LayerConfig("tail", T=T, d=d, F=192, m=48, K=2, way=4, n_shared=1, F_s=Fs, zipf_s=1.0)


def test_sums_launched(tmp_path):
    calls = [dict(entry="forward", cfg=[d, 192, 48, 2, 4, 1, Fs, 0, 0, 0], T=T, threshold=1.0) for T, d, Fs, _, _ in CASES]
    for (T, d, Fs, s1, s2), r in zip(CASES, trace(calls, tmp_path)):
        assert r["status"] == 0
        sums = [l["symbol"] for l in r["launches"] if l["name"] == "gemm_tail_sum_kernel"]
        assert [sum("ILb1E" in s for s in sums), sum("ILb0E" in s for s in sums)] == [s1, s2], (T, d, Fs, sums)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(case):
    T, d, Fs = case[:3]
    print(case, flush=True)
    cfg = _cfg(T, d, Fs)
    L = WL.make_layer(cfg, T, "cpu")
    to = lambda t: tuple(a.to("cuda") for a in t)
    c = P.config_of(cfg)
    ws = P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    got = npf(P.moe_forward(c, L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda"), to(L.experts), None, to(L.shared), 1.0, False,
                            workspace=ws))
    r = oracle_route(L, cfg, 1.0)
    united = WL.make_random_united(cfg, 1, "cpu")         # no row goes to them
    tokens = np.nonzero(r.margin >= 1e-6)[0][::32].astype(np.int32)
    want = O.forward_tokens(npf(L.x), r.topk_idx, r.topk_w, r.expert_unit, cfg.way, npf(L.experts), npf(united), npf(L.shared), tokens=tokens)
    assert np.isfinite(got).all()
    assert rel_err(got[tokens], want) <= OUT_TOL
