"""The trainer's divisions and square root are the correctly rounded ones: one step on one token that is not zero, with the gradients known
exactly, against the same operations in numpy, bit for bit.

Sums stay exact: a product has one term (the other tokens are zero), or three that are the bf16 pieces of one fp32 number.  Weights start at
zero where their update is looked at, so that its bits are the result's.  SwiGLU's results are aimed at the middle between two bf16 numbers and the
step size lies there, so that one ulp of fp32 shows; a gradient near Adam's eps shows its size and not its sign alone."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL

pytestmark = pytest.mark.gpu

N, D, F = 64, 128, 1024
LR = np.float32((1 + 2.0 ** -8) * 2.0 ** -4)
PIECES = (0, 32, 64)                                     # columns of x, a k step of the matrix cores each, that hold a number's pieces
f32 = np.float32


def _bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16)


def _split(v):
    """Three bf16 numbers whose sum is v, added from the first."""
    out, rest = [], np.asarray(v, np.float32)
    for _ in PIECES:
        out.append(_bf16(rest).float().numpy())
        rest = rest - out[-1]
    assert not rest.any()
    return out


def _middle(rng, shape, exponent):
    """Numbers in the middle between two bf16 ones."""
    return np.ldexp((2 * rng.integers(128, 256, shape) + 1) / 256.0, exponent)


def _gates(rng):
    """G, 1 + e^-G and the sigmoid; the rounding of the sum does not hang on the last bits of the exponential."""
    g = rng.uniform(7.0, 12.0, 4 * F).astype(np.float32)
    s = 1.0 + np.exp(-g.astype(np.float64))
    ulps = np.ldexp(s - 1.0, 23)
    keep = np.abs(ulps - np.floor(ulps) - 0.5) > 0.05
    g, s = g[keep][:F], s[keep][:F].astype(np.float32)
    assert len(g) == F
    return g, s, f32(1) / s


def _adam(prod):
    """The update of weights that are zero, first step."""
    b1, b2 = f32(0.9), f32(0.999)
    c1, c2 = f32(1.0 / (1.0 - np.float64(b1))), f32(1.0 / (1.0 - np.float64(b2)))
    gr = prod * f32(2.0 / N)
    m, v = (f32(1) - b1) * gr, (f32(1) - b2) * gr * gr
    return _bf16(f32(0) - LR * (m * c1) / (np.sqrt(v * c2) + f32(1e-8)))


def _train(w1, w3, w2, mean):
    """One step from these weights; `mean`: the teachers' output for the token (both teachers are the same: 32 t y through one column)."""
    cfg = P.config_of(WL.LayerConfig("rounding", T=N, d=D, F=F, m=2, K=1, way=2))
    x = np.zeros((N, D), np.float32)
    x[0, list(PIECES) + [96]] = 1.0
    t1, t3, t2 = (np.zeros(s, np.float32) for s in ((F, D), (F, D), (D, F)))
    t1[0, 0], t3[0, 0], t2[:, 0] = 32.0, 1.0 / 32, mean
    both = tuple(_bf16(np.stack([t, t])).to("cuda") for t in (t1, t3, t2))
    united = tuple(_bf16(w[None]).to("cuda") for w in (w1, w3, w2))
    for u, w in zip(united, (w1, w3, w2)):
        assert np.array_equal(u[0].float().cpu().numpy(), w)            # held in bf16 as they are
    P.moe_distill_united(cfg, both, united, _bf16(x).to("cuda"), 1, float(LR))
    return tuple(u[0].cpu() for u in united)


def _rows(v):
    w = np.zeros((F, D), np.float32)
    for k, piece in zip(PIECES, _split(v)):
        w[:, k] = piece
    return w


def test_forward_and_update():
    rng = np.random.default_rng(1)
    g, s, _ = _gates(rng)
    silu = g / s
    u = (_middle(rng, F, -9) / silu).astype(np.float32)
    a = _bf16(silu * u).float().numpy()
    # columns whose gradients lie around eps, and others where the update is the step size to the last ulp
    mean = np.ldexp(rng.integers(128, 256, D) / 128.0, np.where(np.arange(D) % 2, rng.integers(12, 15, D), -13)).astype(np.float32)
    got = _train(_rows(g), _rows(u), np.zeros((D, F), np.float32), mean)[2]
    want = _adam(-mean[:, None] * a[None, :])
    print("differ:", int((got != want)[::2].sum()), "of small gradients,", int((got != want)[1::2].sum()), "of large ones")
    assert torch.equal(got, want)


def test_backward():
    rng = np.random.default_rng(2)
    g, s, sg = _gates(rng)
    da = (_middle(rng, F, -23) / (g.astype(np.float64) * sg)).astype(np.float32)
    slope = (1.0 + g.astype(np.float64) * (f32(1) - sg)).astype(np.float32)
    u = (_middle(rng, F, -23) / (da.astype(np.float64) * sg * slope)).astype(np.float32)
    w2 = np.zeros((D, F), np.float32)
    for k, piece in zip(PIECES, _split(-da)):
        w2[k] = piece
    mean = np.zeros(D, np.float32)
    mean[list(PIECES)] = 1.0                             # the student's own output there is too small to show beside it
    assert np.abs(w2).sum(1).max() * 32 < 2.0 ** -10
    new = _train(_rows(g), _rows(u), w2, mean)
    for i, grad in ((0, da * u * sg * slope), (1, da * g * sg)):
        got, want = new[i][:, 96], _adam(_bf16(grad).float().numpy())
        print("weights", i, "differ:", int((got != want).sum()), "of", F)
        assert torch.equal(got, want)
