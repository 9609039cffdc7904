"""Divergence importances where their kernels' split of the work can go wrong,
against the oracle: rows about 64 and 256, trees about 8 and the 64 a workgroup
holds in flight, every class-count width, frequencies that are powers of two (their
logarithms end at a digit), blocks of rows, paths to 30 nodes, regression.  All
results are integers or quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,K,trees,depth,kl_rows", [
    (2, 1, 2, 1, 2, 0), (63, 3, 2, 4, 5, 0), (257, 4, 3, 9, 12, 0), (400, 5, 4, 65, 30, 0),
    (300, 6, 7, 33, 9, 64), (520, 3, 13, 8, 12, 257), (700, 2, 3, 130, 3, 1)])
def test_divergence_importances_match_the_oracle(n, p, K, trees, depth, kl_rows):
    rng = np.random.default_rng(40 + n)
    X = np.round(2 * rng.standard_normal((n, p))).astype(np.float32)
    y = np.argmax(X[:, :1] * np.arange(K) + rng.standard_normal((n, K)), axis=1).astype(np.int32)
    kw = dict(max_iter=2, seed=23 + n, n_bins=32, importance_mode=B.PERMUT_KL)
    print(f"divergence n={n} p={p} K={K} T={trees} D={depth} rows={kl_rows}", flush=True)
    o = O.boruta_fit(X, y, K, trees, depth, trace=True, **kw)
    g = B.boruta_fit_ex(X, y, K, trees, depth, trace=True,
                        tune=dict(kl_rows=kl_rows) if kl_rows else None, **kw)
    assert_same_run(g, o)


def test_squared_divergences_match_the_oracle():
    rng = np.random.default_rng(7)
    X = rng.standard_normal((300, 4)).astype(np.float32)
    y = X[:, 0] * 3 + rng.standard_normal(300)
    kw = dict(max_iter=2, seed=9, n_bins=32, importance_mode=B.PERMUT_KL)
    o = O.boruta_fit_reg(X, y, 9, 12, trace=True, **kw)
    assert_same_run(B.boruta_fit_regression(X, y, 9, 12, trace=True, **kw), o)
