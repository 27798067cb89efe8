"""The trainer's workspace on the host: the size never falls as the calibration set grows, what is sized for a large set serves
every smaller one, and workspaces that served when groups were trained one at a time still do.  (Launches go to a stand-in HIP
runtime; that groups side by side give what single ones give is checked on the GPU.)"""
import ctypes as C

import pytest

import paper_2507_17133_amd as P
from paper_2507_17133_amd import binding as B
from tests._fake_hip import trace

#            d, F, m, K, way, n_shared, F_s, score_fn, residual, gate format
SHAPES = {"60 experts": [2048, 1408, 60, 4, 8, 1, 5632, 0, 0, 0], "256 experts": [7168, 2048, 256, 8, 8, 1, 2048, 1, 0, 0],
          "128 experts": [2048, 768, 128, 8, 8, 0, 0, 0, 0, 0], "pairs of large ones": [4096, 14336, 8, 2, 2, 0, 0, 0, 0, 0],
          "small": [256, 512, 8, 2, 8, 0, 0, 0, 0, 0], "ragged": [64, 192, 7, 3, 3, 0, 0, 0, 0, 0],
          "nothing to train": [64, 64, 3, 1, 1, 0, 0, 0, 0, 0]}
# bytes for 64, 512 and 4096 tokens with one group at a time and its gradients in memory: what programs have sized theirs to
ONE_AT_A_TIME = {"60 experts": (160707328, 317780992, 838271488), "256 experts": (791051264, 1048183040, 2105943296),
                 "128 experts": (92820992, 245342720, 528094720), "pairs of large ones": (2976917504, 3278928384, 5028519936),
                 "small": (8230912, 32795648, 141258752), "ragged": (1244928, 13334016, 66017792)}


def _size(shape, n):
    b = C.c_size_t(0)
    assert P.lib().moe_distill_workspace_size(C.byref(B.moe_config(*SHAPES[shape])), n, C.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("shape", SHAPES)
def test_size_never_falls(shape):
    sizes = [_size(shape, n) for n in list(range(64, 9000, 64)) + [16384, 16448, 65536]]
    assert sizes == sorted(sizes)


def test_a_larger_workspace_serves_every_smaller_set(tmp_path):
    def status(calls):
        return [r["status"] for r in trace(calls, tmp_path)]

    call = lambda s, n, b: dict(entry="distill", cfg=SHAPES[s], T=n, steps=1, workspace_bytes=b)
    assert set(status([call(s, n, _size(s, big)) for s in SHAPES for big in (2048, 16384) for n in (64, 128, 512, 960, 2048)])) == {0}
    assert set(status([call(s, n, b) for s, bs in ONE_AT_A_TIME.items() for n, b in zip((64, 512, 4096), bs)])) == {0}
    # not even one group: the forward workspace alone
    assert set(status([call(s, n, P.workspace_size(B.moe_config(*SHAPES[s]), n)) for s in SHAPES for n in (64, 2048)])) == {-4}
