"""Making united experts at the shapes where the batched kernels can go wrong: matrices that end in half a tile,
one slot of FFN rows or several, teachers in several batches, several groups trained side by side, ragged groups."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import distill_oracle as DO
from paper_2507_17133_amd import binding as P
from paper_2507_17133_amd import workloads as WL

DEV = "cuda"

# (n, d, F, m, K, n_shared, way): tiles of 128 with 64 left over in every role; K + n_shared = FFN rows held at a time
SHAPES = [(64, 64, 64, 2, 1, 0, 2), (192, 320, 192, 5, 1, 0, 2), (192, 64, 448, 7, 3, 0, 7), (448, 192, 128, 9, 2, 1, 4),
          (128, 128, 256, 20, 4, 0, 2)]


def f64(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("n,d,F,m,K,ns,way", SHAPES)
def test_loss_and_training_against_the_oracle(n, d, F, m, K, ns, way):
    cfg = WL.LayerConfig("united_shapes", T=n, d=d, F=F, m=m, K=K, way=way, n_shared=ns, F_s=F)
    L = WL.make_layer(cfg, 4, "cpu")
    experts = tuple(t.to(DEV) for t in L.experts)
    x = WL.make_activations(cfg, 4, "cpu", "calib", n)
    c = P.config_of(cfg)
    united, loss = P.moe_build_united(c, experts, x.to(DEV))
    start = [f64(u) for u in united]
    steps, lr = 3, 1e-3
    hist = P.moe_distill_united(c, experts, united, x.to(DEV), steps, lr).cpu().numpy()
    xs = f64(x)
    for g in range(cfg.G):
        lo, hi = g * way, min(m, (g + 1) * way)
        teachers = [tuple(f64(w[i]) for w in L.experts) for i in range(lo, hi)]
        want = DO.loss(xs, tuple(s[g] for s in start), teachers)
        # FFN rows in half precision (2^-11, toward zero: the squares shrink by at most 2^-10) from bf16 H
        # (2^-9 relative, zero-mean over d >= 64 features and n >= 64 tokens)
        assert abs(float(loss[g]) - want) <= 5e-3 * want + 1e-6
        if hi - lo == 1:
            assert (hist[g] == 0).all() and all(torch.equal(u[g], e[lo]) for u, e in zip(united, experts))
            continue
        w_ref, h_ref = DO.distill(xs, tuple(s[g] for s in start), teachers, steps, lr)
        assert np.allclose(hist[g], h_ref, rtol=1e-2), (g, hist[g], h_ref)
        _, grads = DO.loss_and_grads(xs, tuple(s[g] for s in start), teachers)
        for u, b, s0, gr in zip(united, w_ref, start, grads):
            u, s0 = f64(u[g]), s0[g]
            da, db = u - s0, b - s0
            # Adam's first steps have full size whatever the gradient, so a weight whose gradient is rounding noise may end up
            # anywhere; where it is at least half its root mean square, operands rounded to bf16 (2^-9 each) change it by a few
            # per cent, and the normalised step by as much: 15 % of the way, and the weight's own rounding to bf16.  A step left
            # out or taken backwards is off by 100 or 200 %.
            sure = np.abs(gr) >= 0.5 * np.sqrt((gr ** 2).mean())
            assert sure.mean() > 0.4
            assert (np.abs(da - db)[sure] <= 0.15 * lr * steps + 2 ** -8 * np.abs(b)[sure]).all()
            # every 64 x 64 block (the ragged tiles end in one): in a float32 model of the trainer 0.999 at the least
            for i in range(0, u.shape[0], 64):
                for j in range(0, u.shape[1], 64):
                    va, vb = da[i:i + 64, j:j + 64].ravel(), db[i:i + 64, j:j + 64].ravel()
                    assert float(va @ vb / np.sqrt((va @ va) * (vb @ vb))) >= 0.99, (i, j)


# fewer calibration tokens than a tile of 64 rows: either kernel of the small heights
@pytest.mark.parametrize("n,d,F,m,K,ns,way", [(1, 64, 64, 2, 1, 0, 2), (20, 64, 320, 5, 2, 1, 2), (37, 128, 8192, 4, 4, 0, 4)])
def test_loss_of_a_few_tokens(n, d, F, m, K, ns, way):
    cfg = WL.LayerConfig("united_few", T=n, d=d, F=F, m=m, K=K, way=way, n_shared=ns, F_s=F)
    L = WL.make_layer(cfg, 4, "cpu")
    x = WL.make_activations(cfg, 4, "cpu", "calib", n)
    united, loss = P.moe_build_united(P.config_of(cfg), tuple(t.to(DEV) for t in L.experts), x.to(DEV))
    for g in range(cfg.G):
        teachers = [tuple(f64(w[i]) for w in L.experts) for i in range(g * way, min(m, (g + 1) * way))]
        want = DO.loss(f64(x), tuple(f64(u[g]) for u in united), teachers)
        # as above, over n d >= 64 terms instead of 4096
        assert abs(float(loss[g]) - want) <= 2e-2 * want + 1e-6
