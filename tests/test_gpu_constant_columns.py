"""Drawn columns without a valid threshold -- one value, or one bin in most nodes
-- with exact ranking, in the kernels that read an item's counts back at the
chosen bin: node-major and column-major histograms and whole trees, one and
several packed words.  All results are integers or quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tune", [dict(small_rows=2, col_level=64), dict(small_rows=2, col_level=1),
                                  None], ids=["node_major", "column", "whole_trees"])
@pytest.mark.parametrize("K", [2, 3, 6, 13])
def test_exact_ranking_of_columns_without_thresholds(K, tune):
    rng = np.random.default_rng(900 + K)
    X = np.zeros((260, 8), np.float32)
    X[:, 1] = -7.5
    X[:, 2] = rng.random(260) < 0.97
    X[:, 3] = rng.random(260) < 0.03
    X[:, 4] = rng.integers(0, 3, 260)
    y = np.argmax(X[:, 4:5] * np.arange(K) + rng.standard_normal((260, K)), axis=1).astype(np.int32)
    print(f"constant columns K={K} tune={tune}", flush=True)
    kw = dict(max_iter=2, seed=41 + K, n_bins=64, mtry=5, trace=True)
    g = B.boruta_fit_ex(X, y, K, 30, 8, split_rank=B.RANK_EXACT, tune=tune, **kw)
    assert_same_run(g, O.boruta_fit(X, y, K, 30, 8, **kw))
