"""Which tiles the trainer's SwiGLU GEMM gets, seen through a stand-in HIP runtime (no GPU, 256 CUs): the kind that was the faster one by 1.5 to
3.3 % of a step where both were timed, on both sides of the rule and at several K."""
import os

import pytest

from paper_2507_17133_amd import binding as B
from tests._fake_hip import trace

if not os.path.exists(B.LIB_PATH):
    from paper_2507_17133_amd import build as _build
    _build.build()

# d, F, tokens, groups, whether 256 x 192 (the others: 128 x 128)
CASES = [(128, 1536, 1856, 5, 0), (256, 1984, 3904, 2, 0), (512, 1600, 3008, 3, 0), (512, 1984, 3648, 2, 0), (512, 1216, 3520, 2, 0),
         (256, 960, 1536, 6, 0), (1024, 1216, 960, 7, 0), (256, 512, 2048, 5, 1), (2048, 1408, 2048, 2, 1), (2048, 3072, 2048, 1, 1),
         (64, 1024, 1152, 4, 1), (320, 1024, 1088, 4, 1), (2048, 768, 128, 4, 0), (2048, 1024, 1152, 1, 0), (64, 64, 64, 1, 0)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    calls = [dict(entry="distill", cfg=[d, F, 2 * G, 1, 2, 0, 0, 0, 0, 0], T=n, steps=2) for d, F, n, G, _ in CASES]
    return trace(calls, tmp_path_factory.mktemp("fake"))


@pytest.mark.parametrize("i", range(len(CASES)))
def test_tiles(launches, i):
    r = launches[i]
    seen = [l["symbol"] for l in r["launches"] if l["name"] == "distill_gemm_kernel" and "ILi0E" in l["symbol"]]
    assert r["status"] == 0 and len(seen) == 3             # two steps and the last loss, all groups side by side
    assert ["ILi0ELi8ELi6E" in s for s in seen] == [bool(CASES[i][4])] * 3, CASES[i]
