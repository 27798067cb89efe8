"""From how many weights on they are streamed past the caches: more than 288 MiB in the units that hold rows and the shared experts, with the
row lists made inside and brought by the caller.  The kernels' flag is read from the workspace; nothing else may differ."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL
from tests._util import npf

pytestmark = pytest.mark.gpu


def _flag(ws, cnt, off):
    """The word before the routed units' tile table in the workspace."""
    left = ws.cpu().numpy().tobytes()
    for bm in (32, 64, 128, 256):
        tiles = [(u, off[u] + r, min(bm, n - r), 0) for u, n in enumerate(cnt) for r in range(0, int(n), bm)]
        at = left.find(np.asarray([(len(tiles), bm, 0, 0)] + tiles, np.int32).tobytes())
        if at >= 0:
            return int(np.frombuffer(left, np.int32, 1, at - 4)[0])
    raise AssertionError("no table")


# units that may hold rows without their weights being streamed: 24 of 12 MiB are 288 MiB; a shared expert of another width brings 3 MiB
@pytest.mark.parametrize("Fs,below", [(0, 24), (512, 23)])
@pytest.mark.parametrize("T", [40, 150, 700])
def test_both_sides_of_the_line(T, Fs, below):
    print(T, Fs, flush=True)
    m = below + 2
    cfg = WL.LayerConfig("line", T=40 * T, d=1024, F=2048, m=m, K=1, way=4, n_shared=int(Fs > 0), F_s=Fs)
    L = WL.make_layer(cfg, T, "cuda")
    c = P.config_of(cfg)
    of = npf(P.moe_route(c, L.x, L.gate_w, L.gate_b, 1.0).topk_idx)[:, 0]
    pool = [list(np.nonzero(of == e)[0]) for e in range(m)]
    chosen = np.concatenate([pool[e][:T // below + (e < T % below)] for e in range(below)] + [pool[below][:1]])
    assert len(chosen) == T + 1
    x = L.x[torch.as_tensor(chosen, device="cuda")].contiguous()
    outs = {}
    for n in (T, T + 1):                             # one token more, of another unit
        xs = x[:n].contiguous()
        R = P.moe_route(c, xs, L.gate_w, L.gate_b, 1.0)
        assert int((R.unit_cnt[:m] > 0).sum()) == below + (n - T)
        for own in (None, R):
            ws = P.alloc_workspace(c, n)
            ws.fill_(0x5A)
            outs[n, own is None] = P.moe_forward(c, xs, L.gate_w, L.gate_b, L.experts, None, L.shared, 1.0, route=own, workspace=ws)
            torch.cuda.synchronize()
            assert _flag(ws, npf(R.unit_cnt)[:m + cfg.G], npf(R.unit_off)) == n - T
        assert torch.equal(outs[n, True], outs[n, False])
    assert torch.equal(outs[T + 1, True][:T], outs[T, True])
