"""Permutation importances where their kernel's split of the work can go wrong,
against the oracle: out-of-bag rows about a workgroup's 128, trees no multiple of
the 8 XCDs, a row's positions dealt to one to eight workgroups, paths of one node
to 30, columns met twice on a path, replicas across groups of eight pairs, columns
past 16 bits, per-column sums in LDS and not, regression.  All results are integers
or quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,K,trees,depth,n_perm", [
    (2, 1, 2, 9, 1, 1), (12, 3, 2, 8, 3, 2), (345, 4, 3, 7, 30, 3), (360, 2, 4, 17, 12, 9),
    (900, 1100, 2, 3, 9, 1), (60, 33000, 2, 2, 5, 1), (3000, 8, 3, 130, 8, 1),
    (3000, 8, 5, 530, 4, 2)])
def test_permutation_importances_match_the_oracle(n, p, K, trees, depth, n_perm):
    rng = np.random.default_rng(n + p)
    X = rng.standard_normal((n, p)).astype(np.float32)
    y = np.argmax(X[:, :1] * np.arange(K) + rng.standard_normal((n, K)), axis=1).astype(np.int32)
    kw = dict(max_iter=2, seed=17 + n, n_bins=32, importance_mode=B.PERMUT, n_perm=n_perm)
    print(f"permut n={n} p={p} K={K} T={trees} D={depth} R={n_perm}", flush=True)
    o = O.boruta_fit(X, y, K, trees, depth, trace=True, **kw)
    assert_same_run(B.boruta_fit_ex(X, y, K, trees, depth, trace=True, **kw), o)


@pytest.mark.parametrize("n,p,trees,depth,n_perm", [(350, 3, 9, 20, 3), (120, 1200, 2, 6, 1)])
def test_squared_error_increases_match_the_oracle(n, p, trees, depth, n_perm):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, p)).astype(np.float32)
    y = X[:, 0] * 3 + rng.standard_normal(n)
    kw = dict(max_iter=2, seed=n, n_bins=32, importance_mode=B.PERMUT, n_perm=n_perm)
    o = O.boruta_fit_reg(X, y, trees, depth, trace=True, **kw)
    assert_same_run(B.boruta_fit_regression(X, y, trees, depth, trace=True, **kw), o)
