"""Whole trees of 9 to 16 classes -- eight waves a tree, taken at 257 to 512 trees of
few (row, draw) pairs -- and the plans on the other side of that line and of the one
for many rows of 5 to 8 classes, against the oracle.  All results are integers or
quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [B.RANK_FP32, B.RANK_EXACT], ids=["fp32", "exact"])
@pytest.mark.parametrize("n,p,K,trees,depth", [
    (300, 9, 13, 257, 10), (450, 8, 16, 260, 8), (120, 30, 9, 512, 7),  # whole trees
    (460, 8, 16, 257, 8),                                               # past 1,800 pairs
    (2000, 5, 8, 257, 7), (2010, 5, 8, 257, 7)])                        # rows times classes
def test_wide_whole_trees_match_the_oracle(n, p, K, trees, depth, rank):
    rng = np.random.default_rng(870 + n + K)
    X = rng.standard_normal((n, p)).astype(np.float32)
    X[:, 0] = np.round(2 * X[:, 0])
    y = np.argmax(X[:, :1] * np.arange(K) + rng.standard_normal((n, K)), axis=1).astype(np.int32)
    kw = dict(max_iter=2, seed=5 + n, n_bins=64, trace=True)
    print(f"whole trees n={n} p={p} K={K} T={trees} D={depth} rank={rank}", flush=True)
    o = O.boruta_fit(X, y, K, trees, depth, **kw)
    assert_same_run(B.boruta_fit_ex(X, y, K, trees, depth, split_rank=rank, **kw), o)
