"""Which forward calls look at whether their weights are streamed past the caches: none whose TopK entries cannot reach enough units, nor one
whose layer is small.  Seen through a stand-in HIP runtime (no GPU): a template argument of the kernels,
the last one of route_rows_kernel and the one before the last of the GEMMs."""
import os
import re

from paper_2507_17133_amd import binding as B
from tests._fake_hip import trace

if not os.path.exists(B.LIB_PATH):
    from paper_2507_17133_amd import build as _build
    _build.build()

LOOKING = ("route_rows_kernel", "ffn_gemm_kernel", "ffn_gemm_narrow_kernel", "ffn_gemm_either_kernel", "ffn_gemm_pair_kernel", "ffn_gemm_ws_kernel")

#   d, F, m, K, n_shared, F_s, threshold, tokens that cannot stream, tokens that may.  A unit's weights are 6 d F bytes: 0.8 MB; 9.4 MB, one
#   token reaches 8 of them; 17.3 MB beside a shared expert of 69 MB; 352 MB; a shared expert of 617 MB; many rows
SHAPES = [(256, 512, 8, 2, 0, 0, 0.75, (1, 64, 300, 3000), ()),
          (2048, 768, 128, 8, 0, 0, 0.5, (1, 2), (8, 100, 900)),
          (2048, 1408, 60, 4, 1, 5632, 0.4, (1, 2), (16, 37, 300)),
          (2048, 1408, 60, 4, 1, 5632, 1.0, (1, 2), (16, 37, 300)),
          (4096, 14336, 8, 2, 0, 0, 1.0, (), (1, 256)),
          (7168, 256, 8, 2, 1, 14336, 1.0, (), (1, 256)),
          (2048, 768, 128, 8, 0, 0, 0.5, (6144,), (6143,))]         # 384 rows per expert: 256-row tiles, which are not streamed


def test_kernels_that_look(tmp_path):
    calls, want = [], []
    for d, F, m, K, ns, Fs, thr, never, may in SHAPES:
        for own in (0, 1):
            for T in never + may:
                calls.append(dict(entry="forward", cfg=[d, F, m, K, 8, ns, Fs, 0, 0, 0], T=T, threshold=thr, own_route=own))
                want.append(T in may)
    calls += [dict(entry="build", cfg=[2048, 1408, 60, 4, 8, 0, 0, 0, 0, 0], T=300), dict(entry="route", cfg=[4096, 14336, 8, 2, 8, 0, 0, 0, 0, 0], T=40),
              dict(entry="distill", cfg=[2048, 1408, 60, 4, 8, 0, 0, 0, 0, 0], T=64, steps=1)]
    want += [False] * 3
    for c, looks, r in zip(calls, want, trace(calls, tmp_path)):
        assert r["status"] == 0
        seen = [l for l in r["launches"] if l["name"] in LOOKING]
        assert len(seen) >= (1 if c["entry"] == "route" or c["T"] > 2000 else 2) - c.get("own_route", 0), c
        own_width = c["cfg"][5] and c["cfg"][6] != c["cfg"][1]
        gemms = {}
        for l in seen:
            flags = re.findall(r"Lb([01])E", l["symbol"])
            if "route" in l["name"]:
                assert flags[-1:] == [str(int(looks))], (c, l["symbol"])
            else:
                gemms.setdefault(flags[-1], []).append((flags[-2:-1], l))
        for launches in gemms.values():              # GEMM1, GEMM2: routed units first, then shared experts of a width of their own
            for i, (flag, l) in enumerate(launches):
                shared = own_width and i == len(launches) - 1 > 0 and l["name"] != "ffn_gemm_ws_kernel"
                assert flag == [str(int(looks and not shared))], (c, l["symbol"])
        if c.get("own_route"):
            assert [l["grid"] for l in r["launches"] if l["name"] == "tile_table_kernel"] == [(2 if own_width else 1) + looks], c
