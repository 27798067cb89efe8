"""Weights that are streamed past the caches: 21 units of 12.6 MB are not, 22 are (256 MiB), and nothing else may differ.  Units of one tile, of
several and without rows beside each other, at tiles of 32, 64 and 128 rows, with and without a shared expert of a width of its own."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._util import OUT_TOL, check_route, npf, oracle_route, rel_err

pytestmark = pytest.mark.gpu

COUNTS = {30: [1, 2, 1], 150: [40, 1, 33, 2, 32], 700: [150, 129, 1, 128, 64, 65]}      # rows of the first units, the rest get some


@pytest.mark.parametrize("T", list(COUNTS))
@pytest.mark.parametrize("Fs", [0, 192])
def test_streaming_does_not_show(T, Fs):
    print(T, Fs, flush=True)
    below = 21                                       # 192 columns more are 1.2 MB: the line stays between 21 and 22
    cfg = WL.LayerConfig("streamed", T=40 * T, d=1024, F=2048, m=24, K=1, way=4, n_shared=int(Fs > 0), F_s=Fs)
    L = WL.make_layer(cfg, T, "cuda")
    c = P.config_of(cfg)
    of = npf(P.moe_route(c, L.x, L.gate_w, L.gate_b, 1.0).topk_idx)[:, 0]
    pool = [list(np.nonzero(of == e)[0]) for e in range(24)]
    want = COUNTS[T] + [0] * (below - len(COUNTS[T]))
    for k in range(T - sum(want)):                   # the other units by turns
        want[len(COUNTS[T]) + k % (below - len(COUNTS[T]))] += 1
    chosen = np.concatenate([pool[e][:n] for e, n in enumerate(want)])
    assert len(chosen) == T and min(want) > 0
    x = torch.cat([L.x[torch.as_tensor(chosen, device="cuda")], L.x[int(pool[23][0])][None]]).contiguous()
    out = {}
    for tokens in (T, T + 1):                        # one token more, of a 22nd unit
        R = P.moe_route(c, x[:tokens].contiguous(), L.gate_w, L.gate_b, 1.0)
        assert int((R.unit_cnt[:24] > 0).sum()) == below + (tokens - T)
        out[tokens] = P.moe_forward(c, x[:tokens].contiguous(), L.gate_w, L.gate_b, L.experts, None, L.shared, 1.0)
    torch.cuda.synchronize()
    assert torch.equal(out[T + 1][:T], out[T])
    L.x = x
    idx, w, unit = check_route(R, oracle_route(L, cfg, 1.0), cfg, 1.0, False)
    tokens = np.append(np.arange(0, T, 7), T).astype(np.int32)
    ref = O.forward_tokens(npf(x), idx, w, unit, 4, npf(L.experts), None, npf(L.shared), tokens=tokens)
    assert rel_err(npf(out[T + 1])[tokens], ref) <= OUT_TOL
