"""Nodes of weight 65536 and more below the root in column-major levels: the
column-major kernel counts in 16 bits and leaves them to the node-major one by a
list.  Lopsided splits put such nodes on two levels; every class-count width.  All
results are integers or quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [B.RANK_FP32, B.RANK_EXACT], ids=["fp32", "exact"])
@pytest.mark.parametrize("K", [2, 3, 4, 7, 12])
def test_heavy_nodes_of_column_levels_match_the_oracle(K, rank):
    n = 140000
    rng = np.random.default_rng(400 + K)
    X = rng.random((n, 3)).astype(np.float32)
    y = rng.integers(0, K, n)
    y[X[:, 0] < 0.05] = 0  # the best split cuts a twentieth off
    y[(X[:, 1] > 0.97) & (X[:, 0] >= 0.05)] = K - 1
    y = y.astype(np.int32)
    kw = dict(max_iter=1, seed=8 + K, n_bins=64, mtry=5, trace=True)
    print(f"heavy nodes K={K} rank={rank}", flush=True)
    g = B.boruta_fit_ex(X, y, K, 3, 4, split_rank=rank, tune=dict(col_level=1), stats=True, **kw)
    nodes = g["traces"][0]["nodes"]  # tree, heap, feature, threshold, rows, decrease
    heavy = nodes[(nodes[:, 1] > 1) & (nodes[:, 4] >= 65536) & (nodes[:, 2] >= 0)]
    assert len(heavy) >= 3 and len(np.unique(heavy[:, 1])) >= 2
    assert g["stats"].hist_col.launches > 0
    assert_same_run(g, O.boruta_fit(X, y, K, 3, 4, **kw))
