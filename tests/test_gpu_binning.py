"""Thresholds and codes at the edges of the chunked sort: chunk sizes, several
chunks, few distinct values across them, heavy ties, infinities and signed zeros,
and more columns than one coding pass takes.  Codes and threshold bit patterns
equal the oracle's."""
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


def _frame(n, p, seed):
    """Columns of different kinds in turn: tie-free, few values, one dominant value,
    255 to 257 distinct values, extremes of the type, constant."""
    rng = np.random.default_rng(seed)
    X = np.empty((n, p), np.float32)
    for j in range(p):
        kind = j % 8
        if kind == 0:
            X[:, j] = rng.normal(0.0, 1e3, n)
        elif kind == 1:
            X[:, j] = rng.integers(-3, 4, n)
        elif kind == 2:
            X[:, j] = np.where(rng.random(n) < 0.97, 5.0, rng.normal(0.0, 1.0, n))
        elif kind in (3, 4, 5):
            X[:, j] = np.exp(rng.integers(0, 252 + kind, n) * 0.25 - 30.0)
        elif kind == 6:
            X[:, j] = rng.choice(np.array([-np.inf, -3e38, -1e-45, -0.0, 0.0, 1e-45, 3e38, np.inf], np.float32), n)
        else:
            X[:, j] = 7.25
    return X


@pytest.mark.parametrize("n,p,max_bins", [
    (1, 3, 2), (255, 9, 256), (1024, 8, 256), (1025, 9, 255), (2048, 8, 2), (2049, 65, 256), (4097, 8, 17),
    (8192, 8, 256), (8193, 16, 256), (16385, 70, 254), (33000, 70, 100), (70001, 8, 256), (262144, 8, 256),
])
def test_thresholds_and_codes(rf, oracle, n, p, max_bins):
    log(f"binning n={n} p={p} max_bins={max_bins}")
    X = _frame(n, p, n + p)
    d = (np.arange(n) % 7).astype(np.int32)
    codes, binner = rf.aiwc_rf_bin(to_dev(X), to_dev(d), 7, max_bins)
    ob = oracle.bin(X, d, 7, max_bins)
    nb, thr = binner.export()
    assert np.array_equal(nb, ob.n_bins)
    assert np.array_equal(thr.view(np.uint32), ob.thresholds.view(np.uint32))
    assert np.array_equal(codes.cpu().numpy(), ob.codes)
    Y = _frame(301, p, 5)  # the fitted thresholds applied to other rows
    e = np.zeros(301, np.int32)
    again, _ = rf.aiwc_rf_bin(to_dev(Y), to_dev(e), 7, max_bins, binner)
    want = np.stack([np.searchsorted(thr[j, :nb[j] - 1], Y[:, j], side="left") for j in range(p)], axis=1)
    assert np.array_equal(again.cpu().numpy()[:, :p], want)
