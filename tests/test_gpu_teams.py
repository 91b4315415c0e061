"""One-wave teams that share a workgroup's LDS copy of the code matrix (the shape of
deep queues: 64 threads, 5 waves per SIMD), against the oracle node for node."""
import os

import numpy as np
import pytest

from tests._gpu import assert_tree_equal, log, to_dev

pytestmark = pytest.mark.gpu

SHAPE = {"AIWC_RF_GROW_BLOCK": "64", "AIWC_RF_GROW_OCC": "5", "AIWC_RF_BIG_COLS": "4"}


@pytest.fixture
def rf(monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_00156_amd import rf as _rf

    for k, v in SHAPE.items():
        monkeypatch.setenv(k, v)
    return _rf


def _data(C, n, bins, scale, seed):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, bins, (n, C)).astype(np.uint8)
    y = np.clip(scale + 0.3 * scale * rng.normal(0.0, 1.0, n) + 0.02 * codes[:, 0], -64.0, 64.0)
    return codes, y, np.full(C, bins, np.int32)


# bins on both sides of the 7-bit comparison and of one bin per lane; responses of
# three and of four digits (weight x response beyond 24 bits); rows around a
# segment and a wave, and a matrix that just fits and just does not fit the LDS;
# more candidates than one staging chunk; few trees and more than a workgroup's
@pytest.mark.parametrize("C,n,bins,scale,trees,mtry,min_node", [
    (35, 2220, 64, 1.5, 5, 12, 1), (35, 2220, 256, 1.5, 40, 9, 1), (35, 2222, 128, 50.0, 4, 20, 3),
    (9, 700, 129, -50.0, 17, 9, 1), (3, 33, 5, 2.0, 3, 2, 1), (1, 64, 64, 2.0, 2, 1, 1), (80, 900, 64, 2.0, 3, 70, 1),
    (35, 2291, 64, 2.0, 3, 6, 1), (35, 2292, 64, 2.0, 3, 6, 1), (35, 2600, 64, 2.0, 3, 6, 1), (200, 300, 31, 2.0, 2, 9, 2),
])
@pytest.mark.parametrize("wide_sums", ["0", "1"])
def test_teams_match_oracle(rf, oracle, monkeypatch, C, n, bins, scale, trees, mtry, min_node, wide_sums):
    log(f"teams C={C} n={n} bins={bins} scale={scale} trees={trees}")
    monkeypatch.setenv("AIWC_RF_WIDE_SUMS", wide_sums)
    codes, y, nb = _data(C, n, bins, scale, n + C)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                            rf.make_params(trees, mtry, min_node, True, 8))
    li = forest.launch()
    assert (li["block"], li["waves_per_simd"], li["wide_phase"]) == (64, 5, 0)
    of = oracle.fit(codes, nb, y, trees, mtry, min_node, seed=8)
    for t, tree in enumerate(forest.export()):
        assert_tree_equal(tree, of.tree(t), f"tree {t}")


# a fused grid: task groups whose trees part, with a held-out fold
def test_teams_task_groups(rf, oracle):
    log("teams task groups")
    codes, y, nb = _data(21, 1500, 64, 2.0, 3)
    fold = (np.arange(1500) % 3).astype(np.int8)
    combos = [(0, 5, 1), (0, 5, 4), (0, 5, 30), (2, 11, 2), (-1, 5, 9), (0, 5, 4)]
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                            [rf.make_params(20, m, k, True, 6) for _, m, k in combos], to_dev(fold),
                            [f for f, _, _ in combos])
    for i, (f, m, k) in enumerate(combos):
        rows = np.arange(1500) if f < 0 else np.nonzero(fold != f)[0]
        of = oracle.fit(codes, nb, y, 20, m, k, seed=6, train_rows=rows)
        for t, tree in enumerate(forest.export(i)):
            assert_tree_equal(tree, of.tree(t), f"forest {i} tree {t}")


# which kernel ran: a launch of teams has a workgroup per sixteen trees, one of
# one-wave workgroups one per tree.  Around the largest code matrix that fits the
# LDS beside sixteen teams' areas: 163840 - 16 x 5184 - 2560 = 78336 bytes
@pytest.mark.parametrize("C,n,trees,teams", [
    (35, 2220, 40, True), (35, 2238, 17, True), (35, 2239, 17, False), (3, 16000, 33, True),
    (36, 2176, 5, True), (36, 2177, 5, False), (65, 1205, 16, True), (65, 1206, 16, False), (200, 300, 5, False),
])
def test_teams_edge(rf, oracle, C, n, trees, teams):
    log(f"teams edge C={C} n={n} trees={trees} teams={teams}")
    codes, y, nb = _data(C, n, 40, 2.0, n + C)
    mtry = max(1, C // 4)
    params = rf.make_params(trees, mtry, 30, True, 8)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y), params)
    li = forest.launch()
    assert (li["block"], li["waves_per_simd"], li["wide_phase"]) == (64, 5, 0)
    assert li["grid"] == (-(-trees // 16) if teams else trees)
    of = oracle.fit(codes, nb, y, trees, mtry, 30, seed=8)
    for t, tree in enumerate(forest.export()):
        assert_tree_equal(tree, of.tree(t), f"tree {t}")


# one-wave workgroups of five waves per SIMD: twenty fit a CU
def test_one_wave_workgroups_per_cu(rf):
    import torch

    log("one-wave workgroups per CU")
    codes, y, nb = _data(40, 2500, 64, 2.0, 1)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                            rf.make_params(6000, 1, 2000, True, 8))
    li = forest.launch()
    assert (li["block"], li["waves_per_simd"], li["wide_phase"]) == (64, 5, 0)
    assert li["grid"] == 20 * torch.cuda.get_device_properties(0).multi_processor_count
