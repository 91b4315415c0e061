"""Prediction kernels at the edges of their dispatch: rows per workgroup, tree
chunks, row strides and alignments.  Sums of integers and one rounding: the
answers equal the oracle's bit for bit."""
import numpy as np
import pytest

from tests._gpu import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_00156_amd import rf as _rf

    return _rf


def _fitted(rf, oracle, C, n, trees, bins, seed, mtry=None):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, bins, (n, C)).astype(np.uint8)
    y = rng.normal(0.0, 1.0, n)
    nb = np.full(C, bins, np.int32)
    mtry = mtry or max(1, C // 3)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                            rf.make_params(trees, mtry, 2, True, seed))
    return forest, oracle.fit(codes, nb, y, trees, mtry, 2, seed=seed), rng


# rows x trees on both sides of the limits of a workgroup per row (1024 rows, 5 x
# 2^16 pairs), of several (above 1024 trees, 2^18 pairs), of lanes per row (2^19
# pairs, up to 128 trees) and of trees walked one at a time (2^20 pairs), whole and
# broken workgroups of 256 rows, one chunk of trees and many, trees in and out of
# fours; columns with even and odd row strides, and the widest row (255 columns)
@pytest.mark.parametrize("C,trees,rows", [
    (2, 1, (1, 1024, 1025, 1280)), (35, 9, (1, 255, 1023, 1024, 1025, 5000, 58254, 58255)),
    (64, 300, (3, 1000, 1092, 1093, 3495, 3496, 4097)), (65, 1030, (1, 254, 255, 513)), (255, 20, (7, 1024, 1025, 26215)),
    (12, 64, (1025, 8192, 8193)), (9, 1024, (1, 320, 321)), (9, 2100, (1, 124, 125)), (7, 128, (1025, 4096, 4097)), (7, 129, (1025, 4064)), (5, 512, (1024, 1025)), (5, 513, (1025, 2049)),
])
def test_predict_paths(rf, oracle, C, trees, rows):
    import torch

    log(f"predict paths C={C} trees={trees}")
    forest, of, rng = _fitted(rf, oracle, C, 700, trees, 61, C)
    q = rng.integers(0, 256, (max(rows), C)).astype(np.uint8)
    P, yhat = oracle.predict(of, q)
    dq = to_dev(q)
    for n in rows:
        assert np.array_equal(rf.aiwc_rf_predict(forest, dq[:n]).cpu().numpy(), yhat[:n]), n
        lo = trees // 3
        s = rf.aiwc_rf_predict_sum(forest, dq[:n], 0, max(1, lo)).cpu().numpy()
        if lo >= 1:
            s = s + rf.aiwc_rf_predict_sum(forest, dq[:n], lo, trees).cpu().numpy()
        assert np.array_equal(s, P[:n]), n
        # codes that start at an odd address
        flat = torch.empty(n * C + 1, dtype=torch.uint8, device="cuda")
        off = flat[1:].view(n, C)
        off.copy_(dq[:n])
        assert np.array_equal(rf.aiwc_rf_predict(forest, off).cpu().numpy(), yhat[:n]), n


# trees of few and of many leaves (by min.node.size), rows on both sides of the limits
# of each route: a workgroup per row (below and above 1024 rows), several, lanes, a row
# per thread (chunks of the trees, and one chunk for a root alone), staged
ROUTES = [
    (6, 60, 100, 40, (1, 1100, 300000)), (30, 400, 30, 1100, (1, 327, 328, 700, 1117, 1118)),
    (5, 400, 30, 400, (1310, 1311, 2621, 2622, 3072, 3073)), (6, 300, 5, 122, (2950, 5908, 5909, 8594, 8596)),
    (9, 2220, 1, 505, (519, 520, 700)), (9, 2220, 1, 300, (873, 874, 900, 1024, 1025)),
    (7, 9000, 1, 60, (1024, 3549, 3550, 4369, 4370)), (50, 40, 9, 700, (700, 1500, 2048, 3000)),
]


@pytest.mark.parametrize("C,n,min_node,trees,rows", ROUTES)
def test_predict_routes(rf, oracle, C, n, min_node, trees, rows):
    import torch

    log(f"predict routes C={C} n={n} min_node={min_node} trees={trees}")
    rng = np.random.default_rng(n + trees)
    codes = rng.integers(0, 61, (n, C)).astype(np.uint8)
    y = rng.normal(0.0, 1.0, n)
    nb = np.full(C, 61, np.int32)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y),
                            rf.make_params(trees, 3, min_node, True, 6))
    of = oracle.fit(codes, nb, y, trees, 3, min_node, seed=6)
    q = rng.integers(0, 256, (max(rows), C)).astype(np.uint8)
    P, yhat = oracle.predict(of, q)
    dq = to_dev(q)
    for k in rows:
        assert np.array_equal(rf.aiwc_rf_predict(forest, dq[:k]).cpu().numpy(), yhat[:k]), k
        out = torch.empty(k, dtype=torch.float64, device="cuda")
        assert np.array_equal(rf.aiwc_rf_predict_noalloc(forest, dq[:k], out).cpu().numpy(), yhat[:k]), k
        assert np.array_equal(rf.aiwc_rf_predict_sum(forest, dq[:k], 0, trees).cpu().numpy(), P[:k]), k


# (kernel, device) rows below and above the per-row kernel's limit
@pytest.mark.parametrize("D,m,trees", [(1, 5, 30), (15, 4, 30), (15, 68, 30), (15, 69, 30), (32, 100, 30), (15, 4, 1100)])
def test_select_paths(rf, oracle, D, m, trees):
    log(f"select paths D={D} m={m} trees={trees}")
    rng = np.random.default_rng(D + m)
    n, C = 600, 12
    codes = rng.integers(0, 40, (n, C)).astype(np.uint8)
    codes[:, -1] = rng.integers(0, D, n)
    nb = np.array([40] * (C - 1) + [D], np.int32)
    y = rng.normal(0.0, 1.0, n)
    forest = rf.aiwc_rf_fit(to_dev(codes), rf.aiwc_rf_binner_from_counts(nb), to_dev(y), rf.make_params(trees, 5, 3, True, 4))
    of = oracle.fit(codes, nb, y, trees, 5, 3, seed=4)
    feat = rng.integers(0, 40, (m, C - 1)).astype(np.uint8)
    best, times = rf.aiwc_rf_select_device(forest, to_dev(feat), n_devices=D)
    rows = np.concatenate([np.repeat(feat, D, axis=0), np.tile(np.arange(D, dtype=np.uint8), m)[:, None]], axis=1)
    _, yhat = oracle.predict(of, rows)
    yhat = yhat.reshape(m, D)
    assert np.array_equal(times.cpu().numpy(), yhat)
    assert np.array_equal(best.cpu().numpy(), yhat.argmin(axis=1))


# training rows around a bitmap word and a workgroup's 512 rows, one and several
# tree chunks, rows too wide for 512 of them, and a forest without bootstrap
@pytest.mark.parametrize("C,n,trees,boot", [
    (35, 2, 3, True), (35, 63, 9, True), (35, 64, 1, True), (34, 65, 40, True), (35, 511, 8, True), (35, 512, 9, True),
    (35, 513, 70, True), (3, 1025, 300, True), (255, 700, 20, True), (35, 600, 10, False),
])
def test_oob_paths(rf, oracle, C, n, trees, boot):
    log(f"oob paths C={C} n={n} trees={trees}")
    rng = np.random.default_rng(n + C)
    codes = rng.integers(0, 61, (n, C)).astype(np.uint8)
    y = rng.normal(0.0, 1.0, n)
    nb = np.full(C, 61, np.int32)
    mtry = max(1, C // 4)
    dc, dy = to_dev(codes), to_dev(y)
    forest = rf.aiwc_rf_fit(dc, rf.aiwc_rf_binner_from_counts(nb), dy, rf.make_params(trees, mtry, 2, boot, 9))
    res = rf.aiwc_rf_oob_error(forest, dc, dy, n_train=n)
    of = oracle.fit(codes, nb, y, trees, mtry, 2, seed=9, bootstrap=boot)
    P, cnt, (_, _, m) = oracle.oob(of, codes, y, mtry, 2, seed=9, bootstrap=boot)
    assert np.array_equal(res.sums.cpu().numpy(), P)
    assert np.array_equal(res.counts.cpu().numpy(), cnt)
    assert res.rows[0] == m


# held-out rows of folds of very different sizes, one of them a single row and one
# above a workgroup's rows, each under all of its forest's trees
@pytest.mark.parametrize("sizes,trees", [((1, 64, 200), 7), ((600, 3, 513), 33)])
def test_heldout_paths(rf, oracle, sizes, trees):
    log(f"heldout paths {sizes}")
    rng = np.random.default_rng(trees)
    n, C = sum(sizes) + 40, 21
    fold = rng.permutation(np.repeat(np.arange(-1, len(sizes)), (40,) + sizes)).astype(np.int8)
    codes = rng.integers(0, 50, (n, C)).astype(np.uint8)
    y = rng.normal(0.0, 1.0, n)
    nb = np.full(C, 50, np.int32)
    dc, dy = to_dev(codes), to_dev(y)
    forest = rf.aiwc_rf_fit(dc, rf.aiwc_rf_binner_from_counts(nb), dy,
                            [rf.make_params(trees + k, 6, 2, True, 5) for k in range(len(sizes))], to_dev(fold),
                            list(range(len(sizes))))
    res = rf.aiwc_rf_heldout_error(forest, dc, dy, n_heldout=sum(sizes))
    sums, at = res.sums.cpu().numpy(), 0
    for k, size in enumerate(sizes):
        of = oracle.fit(codes, nb, y, trees + k, 6, 2, seed=5, train_rows=np.nonzero(fold != k)[0])
        P, yhat = oracle.predict(of, codes[fold == k])
        assert np.array_equal(sums[at:at + size], P), k
        e = yhat - y[fold == k]
        assert res.rows[k] == size
        # n non-negative terms summed in two orders: within 2 n 2^-53 of each other
        assert abs(res.mse[k] - (e * e).mean()) <= 2 * (size + 1) * 2.0 ** -53 * (e * e).mean()
        at += size


# few trees: waves that share a tree's rows (8, 4 and 2 of them, some without rows),
# and workgroups of few rows
@pytest.mark.parametrize("n,forests,trees", [(2200, 130, 1), (2200, 130, 2), (1500, 100, 3), (2200, 130, 5), (300, 3, 1),
                                             (9000, 1, 1), (9000, 1, 4), (9000, 2, 11)])
def test_scores_of_few_trees(rf, oracle, n, forests, trees):
    log(f"scores of few trees n={n} forests={forests} trees={trees}")
    rng = np.random.default_rng(n + trees)
    C = 13
    codes = rng.integers(0, 61, (n, C)).astype(np.uint8)
    y = rng.normal(0.0, 1.0, n)
    nb = np.full(C, 61, np.int32)
    fold = rng.integers(0, 2, n).astype(np.int8)
    dc, dy = to_dev(codes), to_dev(y)
    forest = rf.aiwc_rf_fit(dc, rf.aiwc_rf_binner_from_counts(nb), dy,
                            [rf.make_params(trees, 4, 3, True, 20 + k) for k in range(forests)], to_dev(fold),
                            [k % 2 for k in range(forests)])
    sums, counts, held = [], [], []
    for k in range(forests):
        rows = np.nonzero(fold != k % 2)[0]
        of = oracle.fit(codes, nb, y, trees, 4, 3, seed=20 + k, train_rows=rows)
        P, cnt, _ = oracle.oob(of, codes, y, 4, 3, seed=20 + k, train_rows=rows)
        sums.append(P)
        counts.append(cnt)
        held.append(oracle.predict(of, codes[fold == k % 2])[0])
    res = rf.aiwc_rf_oob_error(forest, dc, dy, n_train=sum(len(P) for P in sums))
    assert np.array_equal(res.sums.cpu().numpy(), np.concatenate(sums))
    assert np.array_equal(res.counts.cpu().numpy(), np.concatenate(counts))
    res = rf.aiwc_rf_heldout_error(forest, dc, dy, n_heldout=sum(len(P) for P in held))
    assert np.array_equal(res.sums.cpu().numpy(), np.concatenate(held))


# node arrays taken tree by tree (up to four trees) and unpacked on the device
def test_export_few_and_many(rf, oracle):
    log("export few and many trees")
    forest, of, _ = _fitted(rf, oracle, 9, 400, 7, 30, 2)
    for a, b in ((0, 1), (2, 6), (1, 6), (0, 7)):
        for t, tree in zip(range(a, b), forest.export(0, a, b)):
            ot = of.tree(t)
            for k in ("col", "bin", "left", "q", "N"):
                assert np.array_equal(tree[k], ot[k]), (a, b, t, k)
