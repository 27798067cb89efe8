"""Training that meets numbers which are not finite says so: NaN or infinity among the calibration tokens, and a step size
with which the weights overflow, show in the loss history and in no other group's."""
import numpy as np
import pytest
import torch

import paper_2507_17133_amd as P
from paper_2507_17133_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _train(calib, lr, steps):
    cfg = WL.LayerConfig("nonfinite", T=128, d=128, F=192, m=5, K=2, way=2)
    L = WL.make_layer(cfg, 0, "cpu")
    experts = tuple(a.to("cuda") for a in L.experts)
    c = P.config_of(cfg)
    united, _ = P.moe_build_united(c, experts)
    return P.moe_distill_united(c, experts, united, calib.to("cuda"), steps, lr).cpu().numpy()


def _calib():
    return WL.make_activations(WL.LayerConfig("nonfinite", T=128, d=128, F=192, m=5, K=2, way=2), 0, "cpu", "calib", 192)


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("steps", [0, 2])
def test_a_calibration_token_that_is_not_finite(value, steps):
    x = _calib()
    x[70, 3] = value
    hist = _train(x, 1e-3, steps)
    assert not np.isfinite(hist[:2]).any(), hist
    assert (hist[2] == 0).all()                       # one member: not trained


def test_a_step_size_that_overflows_the_weights():
    hist = _train(_calib(), 1e30, 3)
    assert np.isfinite(hist[:2, 0]).all() and not np.isfinite(hist[:2, 1:]).any(), hist
    assert (hist[2] == 0).all()
