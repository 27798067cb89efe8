"""Workspaces that programs have sized once and kept: what the size query gave for these layers stays enough."""
import pytest

import paper_2507_17133_amd as P

KEPT = [(P.make_config(2048, 1408, 60, 4, 8, 1, 5632), {37: 8794880, 1021: 212040192, 4096: 438238208}),
        (P.make_config(7168, 2048, 256, 8, 8, 1, 2048, 1), {37: 32543232, 1021: 256508928, 4096: 759569408}),
        (P.make_config(2048, 768, 128, 8, 8), {37: 7287040, 1021: 215648768, 4096: 256512000}),
        (P.make_config(4096, 14336, 8, 2, 2), {37: 11892224, 1021: 199961088, 4096: 448335872}),
        (P.make_config(256, 512, 8, 2, 8), {37: 495104, 1021: 23364096, 4096: 69691904}),
        (P.make_config(64, 192, 7, 3, 3), {37: 203520, 1021: 15499008, 4096: 42857472}),
        (P.make_config(4096, 4096, 64, 8, 8), {37: 15807232, 1021: 276294144, 4096: 608399872})]


@pytest.mark.parametrize("cfg,sizes", KEPT)
def test_sizes_have_not_grown(cfg, sizes):
    for T, n in sizes.items():
        assert P.workspace_size(cfg, T) <= n, T
