"""Tile heights that the device chooses from the row counts within one launch: 32 or 64 rows and 64 or 128, with even and skewed gates, with
and without brownout, with shared experts of the same width, beside shared experts of another, and where a third height has a launch
of its own.  The table left in the workspace has the height that saves rounds of blocks; a route brought by the caller takes
the same one; outputs against the oracle."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._util import OUT_TOL, check_route, npf, oracle_route, rel_err

pytestmark = pytest.mark.gpu

MODES = [(1.0, False), (0.6, False), (0.3, True)]
N_CU = 256


def _tiles(cnt, bm):
    return int((-(-cnt // bm)).sum())


def _height(cnt, lo, d, F, planes):
    """GEMM1 has ceil(F / 128) blocks per tile with d / 64 k tiles of two matrices, GEMM2 ceil(d / 256) in each plane with a share of
    the F / 64; the taller height has to save 1 / 13 of the rounds (128 rows) or 1 / 25 (64)."""
    c1, c2, k1, k2 = -(-F // 128), -(-d // 256) * planes, d // 64, -(-(F // 64) // planes)
    cost = lambda n: 2 * -(-n * c1 // N_CU) * k1 + -(-n * c2 // N_CU) * k2
    n, n_lo, own = _tiles(cnt, 2 * lo), _tiles(cnt, lo), 12 if lo == 64 else 24
    return 2 * lo if (lo == 64 and 2 * n * c1 <= N_CU) or (own + 1) * cost(n) <= own * cost(n_lo) else lo


def _planes(T, d, F, m, K, G, ns):
    rows = T * K // m
    bm = 64 if rows >= 24 else 32
    tiles = (T * (K + ns) // bm + (m + G) // 2 + ns) * -(-d // 256)
    ks = 1
    while ks < 4 and tiles * ks < 1024 and F // 64 // (2 * ks) >= 8:
        ks *= 2
    return ks


def _table(cnt, off, bm):
    tiles = [(u, off[u] + r, min(bm, cnt[u] - r), 0) for u in range(len(cnt)) for r in range(0, int(cnt[u]), bm)]
    return np.asarray([(len(tiles), bm, 0, 0)] + tiles, np.int32).tobytes()


# T, d, F, m, K, n_shared, F_s, zipf, the lower height; the height taken in each of MODES
CASES = [(44, 1024, 1664, 20, 2, 0, 0, None, 32, (32, 32, 32)), (110, 1024, 1664, 20, 2, 0, 0, 1.2, 32, (64, 32, 32)),
         (66, 1088, 576, 60, 4, 1, 576, 1.0, 32, (32, 32, 32)), (70, 1024, 1472, 24, 3, 1, 192, 1.2, 32, (32, 32, 32)),
         (300, 1024, 4096, 64, 2, 0, 0, 1.0, 32, (32, 64, 64)), (100, 1088, 2112, 24, 2, 1, 320, 0.8, 32, (32, 64, 32)),
         (130, 1024, 1664, 20, 2, 0, 0, None, 64, (64, 64, 128)), (301, 1024, 1664, 20, 2, 0, 0, 1.2, 64, (64, 128, 128)),
         (403, 1088, 576, 60, 4, 1, 576, 1.0, 64, (64, 64, 128)), (300, 1024, 2048, 40, 4, 0, 0, 1.2, 64, (128, 64, 128)),
         (1030, 1024, 8192, 22, 1, 0, 0, 0.7, 64, (128, 128, 256))]            # 256 rows offered


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("mode", range(len(MODES)))
def test_height(case, mode):
    T, d, F, m, K, Ns, Fs, zipf, lo, taken = case
    threshold, full = MODES[mode]
    print(case, mode, flush=True)
    cfg = WL.LayerConfig("rounds", T=T, d=d, F=F, m=m, K=K, way=4, n_shared=Ns, F_s=Fs, zipf_s=zipf)
    L = WL.make_layer(cfg, T + m, "cpu")
    to = lambda t: None if t is None else tuple(a.to("cuda") for a in t)
    x, gate_w, gate_b = L.x.to("cuda"), L.gate_w.to("cuda"), None if L.gate_b is None else L.gate_b.to("cuda")
    united_cpu = WL.make_random_united(cfg, 1, "cpu")
    experts, united, shared = to(L.experts), to(united_cpu), to(L.shared)
    c = P.config_of(cfg)
    ws, ws_r = P.alloc_workspace(c, T), P.alloc_workspace(c, T)
    ws.fill_(0x5A)
    ws_r.fill_(0x5A)
    out = P.moe_forward(c, x, gate_w, gate_b, experts, united, shared, threshold, full, workspace=ws)
    R = P.moe_route(c, x, gate_w, gate_b, threshold, full)
    out_r = P.moe_forward(c, x, gate_w, gate_b, experts, united, shared, route=R, workspace=ws_r)
    torch.cuda.synchronize()
    assert torch.equal(out, out_r)
    units = m + cfg.G + (Ns if Fs == F else 0)
    cnt, off = npf(R.unit_cnt)[:units].astype(int), npf(R.unit_off)
    if taken[mode] <= 2 * lo:
        assert _height(cnt, lo, d, F, _planes(T, d, F, m, K, cfg.G, Ns)) == taken[mode]
    for w in (ws, ws_r):
        left = w.cpu().numpy().tobytes()
        assert [bm for bm in (lo, 2 * lo, 256) if _table(cnt, off, bm) in left] == [taken[mode]]
    idx, w, unit = check_route(R, oracle_route(L, cfg, threshold, full), cfg, threshold, full)
    tokens = np.unique(np.linspace(0, T - 1, 64).astype(np.int32))
    want = O.forward_tokens(npf(L.x), idx, w, unit, 4, npf(L.experts), npf(united_cpu), npf(L.shared), tokens=tokens)
    got = npf(out)
    assert np.isfinite(got).all()
    assert rel_err(got[tokens], want) <= OUT_TOL
