"""Where the row kernel takes the tokens of an expert from: bitmaps of the launch that takes TopK wherever its blocks have 16 tokens,
the TopK lists of at most 16 experts up to 2048 tokens, the routing block's own TopK of a segment of up to 64 experts or of 24 or
32 tokens; with long lists of few experts, which need no more time than the three launches of larger batches."""
import re

import pytest

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._fake_hip import trace
from tests._util import check_route, oracle_route

BITS, LISTS, TOPK, THREE = "0", "1", "2", None
# T, m, K and the source
CASES = [(64, 16, 16, TOPK), (65, 16, 16, LISTS), (100, 1, 1, LISTS), (703, 16, 9, LISTS), (2048, 13, 13, LISTS), (2049, 16, 16, BITS),
         (2065, 3, 2, BITS), (3007, 9, 8, BITS), (8192, 12, 12, BITS), (8193, 16, 8, THREE), (65, 17, 8, BITS), (8192, 40, 17, BITS),
         (64, 64, 15, TOPK), (65, 64, 15, BITS), (64, 65, 1, BITS), (32, 128, 8, TOPK), (33, 65, 15, BITS), (24, 256, 32, TOPK),
         (24, 129, 15, TOPK), (25, 256, 15, BITS), (24, 17, 16, TOPK), (25, 17, 16, BITS), (49, 200, 31, BITS)]


def _source(launches):
    rows = [l["symbol"] for l in launches if l["name"] == "route_rows_kernel"]
    return re.search(r"ILi(\d+)E", rows[0]).group(1) if rows else None


def test_sources_of_the_cases(tmp_path):
    calls = [dict(entry=e, cfg=[128, 64, m, K, 4, 0, 0, 0, 0, f], T=T, threshold=0.5) for T, m, K, _ in CASES
             for e in ("route", "forward", "route_static") for f in (0, 1)]
    want = [c[3] for c in CASES for _ in range(6)]
    for c, w, r in zip(calls, want, trace(calls, tmp_path)):
        assert r["status"] == 0 and _source(r["launches"]) == w, (c, w)


def test_logits_that_fit_the_scratch_go_through_it_at_once(tmp_path):
    """Room for 26 and for 100 tokens or a few more: more than a multiple of 16 or 64, and all there are."""
    calls = [dict(entry=e, cfg=[1024, 64, 256, 2, 8, 0, 0, 0, 0, 1], T=T) for T in (24, 25, 100) for e in ("route", "forward")]
    for c, r in zip(calls, trace(calls, tmp_path)):
        assert r["status"] == 0 and [l["T"] for l in r["launches"] if l["name"] == "gate_logits_kernel"] == [c["T"]], c


@pytest.mark.gpu
@pytest.mark.parametrize("T,m,K", [c[:3] for c in CASES])
@pytest.mark.parametrize("threshold,full", [(1.0, False), (0.4, False), (0.0, True)])
def test_against_the_oracle(T, m, K, threshold, full):
    print(T, m, K, threshold, full, flush=True)
    cfg = WL.LayerConfig("source", T=T, d=128, F=64, m=m, K=K, way=4, n_shared=1, F_s=64, zipf_s=1.0)
    L = WL.make_layer(cfg, T + m, "cpu")
    R = P.moe_route(P.config_of(cfg), L.x.to("cuda"), L.gate_w.to("cuda"), L.gate_b.to("cuda"), threshold, full)
    check_route(R, oracle_route(L, cfg, threshold, full), cfg, threshold, full)
