"""The host code's launches, seen through a stand-in HIP runtime (no GPU): every launch that fails ends its call with an error,
and no kernel runs on what the failed one should have written."""
import os

from paper_2507_17133_amd import binding as B
from tests._fake_hip import trace

if not os.path.exists(B.LIB_PATH):
    from paper_2507_17133_amd import build as _build
    _build.build()

#       d, F, m, K, way, n_shared, F_s, score_fn, residual, gate format
CFGS = {"few": [256, 512, 8, 2, 4, 0, 0, 0, 0, 0], "many": [1024, 256, 60, 4, 8, 1, 512, 0, 0, 0],
        "packed": [1024, 256, 256, 8, 8, 1, 256, 0, 0, 1], "wide": [512, 1024, 40, 20, 4, 0, 0, 0, 0, 1]}
CALLS = [dict(entry=e, cfg=c, T=T, threshold=thr) for e in ("route", "route_static", "forward") for c in CFGS.values()
         for T in (3, 700, 3000) for thr in (1.0, 0.4)]
CALLS = [c for c in CALLS if not (c["entry"] == "route_static" and c["cfg"] is CFGS["wide"] and c["T"] == 3000)]
CALLS += [dict(entry="forward", cfg=CFGS["few"], T=3000, own_route=1), dict(entry="build", cfg=CFGS["many"], T=400),
          dict(entry="distill", cfg=CFGS["few"], T=128, steps=2)]


def test_every_failing_launch_ends_its_call(tmp_path):
    whole = trace(CALLS, tmp_path)
    broken, where = [], []
    for c, r in zip(CALLS, whole):
        assert r["status"] == 0 and len(r["launches"]) >= 2, c
        for k in range(len(r["launches"])):
            broken.append(dict(c, fail=k))
            where.append(r["launches"][k]["name"])
    for c, name, r in zip(broken, where, trace(broken, tmp_path)):
        assert r["status"] == -6, (name, c)
        if name.startswith(("gate_", "prep_")):
            after = [l["name"] for l in r["launches"][c["fail"] + 1:]]
            assert not any(n.startswith(("route_", "ffn_", "combine")) for n in after), (name, after, c)


def test_slices_of_the_gate_do_not_depend_on_the_scratch(tmp_path):
    """The order in which a logit is added up: the same number of K slices in moe_route, moe_forward and every piece of
    moe_route_static."""
    calls = [dict(entry=e, cfg=[d, 256, m, 4, 8, 0, 0, 0, 0, 1], T=T) for d, m in ((7168, 256), (2048, 128), (2048, 60), (1088, 200), (64, 17))
             for T in (1, 40, 300, 1021, 2048, 4999, 8192) for e in ("route", "forward", "route_static")]
    got = trace(calls, tmp_path)
    several = 0
    for c, r in zip(calls, got):
        assert r["status"] == 0
        pieces = [l for l in r["launches"] if l["name"].startswith("gate_logits")]
        assert sum(l["T"] for l in pieces) == c["T"]
        if c["entry"] == "route":
            want = pieces[0]["n_slice"]
        assert {l["n_slice"] for l in pieces} == {want}, c
        several += want > 1 and len(pieces) > 1
    assert several >= 3


def _planes(d, F, m, K, way, ns, T):
    """K slices of GEMM2, whose partial sums are held in half precision: until 1024 tiles of the height that the mean number of
    rows asks for, slices of at least eight k tiles."""
    rows = T * K // m
    bm = 256 if rows >= 384 else 128 if rows >= 48 else 64 if rows >= 24 else 32
    tiles = (T * (K + ns) // bm + (m + -(-m // way)) // 2 + ns) * -(-d // 256)
    ks = 1
    while ks < 4 and tiles * ks < 1024 and F // 64 // (2 * ks) >= 8:
        ks *= 2
    return 1 if bm == 256 else ks


def test_planes_of_partial_sums(tmp_path):
    shapes = [(4096, 4096, 64, 8, 8, 0), (2048, 1408, 60, 4, 8, 1), (4096, 14336, 8, 2, 8, 0), (2048, 768, 128, 8, 8, 0),
              (7168, 2048, 256, 8, 8, 1), (2048, 2048, 40, 4, 4, 0), (256, 512, 8, 2, 8, 0)]
    calls = [dict(entry="forward", cfg=[d, F, m, K, way, ns, F if ns else 0, 0, 0, 0], T=T, threshold=thr)
             for d, F, m, K, way, ns in shapes for T in (1, 20, 64, 96, 112, 150, 191, 230, 384, 900, 2048, 5000) for thr in (1.0, 0.5)]
    for c, r in zip(calls, trace(calls, tmp_path)):
        assert r["status"] == 0 and r["launches"][-1]["planes"] == _planes(*c["cfg"][:6], c["T"]), c


def test_calibration_batches_choose_their_kernel_by_their_own_units(tmp_path):
    """A student and a teacher of 20 tokens at F = 4096 are 2 x 32 blocks of 256 columns in GEMM1, too few for 256 CUs, a student
    and its eight teachers are 288; GEMM2 (d = 256) has a block per unit."""
    calls = [dict(entry="build", cfg=[256, 4096, 8, K, 8, ns, 4096 if ns else 0, 0, 0, 0], T=20) for K, ns in ((2, 0), (8, 8))]
    for c, r, wide in zip(calls, trace(calls, tmp_path), (False, True)):
        gemms = [l["name"] for l in r["launches"] if l["name"].startswith("ffn_gemm")]
        assert r["status"] == 0
        if wide:
            assert gemms[0] == "ffn_gemm_kernel" and gemms[1] == "ffn_gemm_narrow_kernel"
        else:
            assert set(gemms) == {"ffn_gemm_narrow_kernel"}
