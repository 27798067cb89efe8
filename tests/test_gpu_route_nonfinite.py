"""Tokens for which TopK has too few numbers to choose from (a token of NaN; a bias of -infinity that leaves fewer than K
experts): it then names an expert several times.  The counts stay counts of entries, in every batch size, and such an expert's
one row keeps the weight of its last entry."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from oracle import oracle as O
from paper_2507_17133_amd import workloads as WL
from tests._util import npf

pytestmark = pytest.mark.gpu


# 3 tokens: the block that takes TopK routes them; more: a block per 64 tokens counts entries again where tokens name an expert twice
@pytest.mark.parametrize("T,m,K", [(3, 20, 4), (300, 130, 8), (700, 40, 13), (1024, 60, 5), (1100, 60, 5)])
@pytest.mark.parametrize("what", ["nan", "bias"])
@pytest.mark.parametrize("threshold", [1.0, 0.5])
def test_counts_and_rows(T, m, K, what, threshold):
    print(T, m, K, what, threshold, flush=True)
    way, ns = 4, 1
    cfg = WL.LayerConfig("nonfinite", T=T, d=64, F=64, m=m, K=K, way=way, n_shared=ns, F_s=64)
    L = WL.make_layer(cfg, T + m, "cpu")
    x, bias = L.x.clone(), torch.zeros(m)
    if what == "nan":
        x[T // 2] = float("nan")
    else:
        bias[[e for e in range(m) if e not in (0, 7)]] = float("-inf")
    c = P.config_of(cfg)
    R = P.moe_route(c, x.to("cuda"), L.gate_w.to("cuda"), bias.to("cuda"), threshold)
    torch.cuda.synchronize()
    idx, w = npf(R.topk_idx), npf(R.topk_w)
    assert ((idx >= 0) & (idx < m)).all()
    assert any(len(set(r)) < K for r in idx.tolist())             # the case this test is about
    cnt = np.bincount(idx.ravel(), minlength=m)
    assert (npf(R.expert_cnt) == cnt).all()
    unit, s1 = O.brownout_decide(cnt.astype(np.int32), way, threshold, False)
    assert (npf(R.expert_unit) == unit).all() and (npf(R.expert_in_s1) == s1).all()
    U, G = m + (m + way - 1) // way + ns, (m + way - 1) // way
    of = unit[idx]
    rows = [sorted({t for t in range(T) if u in of[t]}) for u in range(m + G)] + [list(range(T))] * ns
    assert (npf(R.unit_cnt) == [len(r) for r in rows]).all()
    off = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    assert (npf(R.unit_off) == off).all() and int(npf(R.n_rows)[0]) == off[U]
    row_token, row_weight, token_rows = npf(R.row_token), npf(R.row_weight), npf(R.token_rows)
    assert (row_token[:off[U]] == np.concatenate([np.asarray(r, np.int64) for r in rows])).all()
    place = [{t: off[u] + i for i, t in enumerate(r)} for u, r in enumerate(rows)]
    for t in range(T):
        for j in range(K):
            u = of[t, j]
            same = [q for q in range(K) if of[t, q] == u]
            row = place[u][t]
            assert token_rows[t, j] == (row if u < m or j == same[0] else -1), (t, j)
            if u < m:
                want = w[t, same[-1]]
            else:
                want = w[t, same[0]]
                for q in same[1:]:
                    want = np.float32(want + w[t, q])
            got = row_weight[row]
            assert got == want or (np.isnan(got) and np.isnan(want)), (t, j, got, want)
