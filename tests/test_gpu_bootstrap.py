"""The bootstrap's counting passes over the LDS, against the oracle: 16- and 32-bit
counters, one pass and several, and the in-bag bitmaps that the passes write."""
import numpy as np
import pytest

from tests._gpu import assert_tree_equal, log, to_dev

pytestmark = pytest.mark.gpu


def _data(n, C, bins, seed):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, bins, (n, C)).astype(np.uint8)
    return codes, rng.normal(0.0, 1.0, n) + 0.1 * codes[:, 0], np.full(C, bins, np.int32)


# the last size of 16-bit counters and its neighbours (one pass of a 1024-thread
# workgroup), sizes that are a whole number of passes and one row more, and
# narrow workgroups, whose area holds fewer rows (one-wave teams: about 2400)
@pytest.mark.parametrize("n,block,occ", [
    (65535, "1024", "4"), (65536, "1024", "4"), (65537, "1024", "4"), (98305, "1024", "4"), (131074, "512", "4"),
    (20001, "192", "4"), (16383, "128", "4"), (9000, "64", "5"), (30001, "64", "4"),
])
@pytest.mark.parametrize("bootstrap", [True, False])
def test_bootstrap_passes(oracle, monkeypatch, n, block, occ, bootstrap):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_00156_amd import rf

    log(f"bootstrap passes n={n} block={block} bootstrap={bootstrap}")
    monkeypatch.setenv("AIWC_RF_GROW_BLOCK", block)
    monkeypatch.setenv("AIWC_RF_GROW_OCC", occ)
    if block in ("64", "128"):
        monkeypatch.setenv("AIWC_RF_HUGE_MIN", str(1 << 18))
    codes, y, nb = _data(n, 4, 16, n)
    min_node = n // 40  # few levels: the test is of the root
    d_codes = to_dev(codes)
    f = rf.aiwc_rf_fit(d_codes, rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                       rf.make_params(3, 2, min_node, bootstrap, 12))
    of = oracle.fit(codes, nb, y, 3, 2, min_node, bootstrap=bootstrap, seed=12)
    for t, tree in enumerate(f.export()):
        assert_tree_equal(tree, of.tree(t), f"tree {t}")
    res = rf.aiwc_rf_oob_error(f, d_codes, to_dev(y), n_train=n)
    P, cnt, (_, _, m) = oracle.oob(of, codes, y, 2, min_node, seed=12, bootstrap=bootstrap)
    assert res.rows[0] == m
    assert np.array_equal(res.sums.cpu().numpy(), P)
    assert np.array_equal(res.counts.cpu().numpy(), cnt)
