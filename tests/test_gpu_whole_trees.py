"""Trees grown whole by one workgroup each (the library's choice for few trees of
few rows) against the oracle, and against the level kernels that a chosen launch
shape selects: roots that are leaves, small and large nodes, every class-count
width, both rankings, draws past one round of 64, several jobs, graph replay and
eager launches.  All results are integers or quotients of them: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


def problem(seed, n, p, K):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, p)).astype(np.float32)
    X[:, 0] = np.round(2 * X[:, 0])
    y = np.argmax(X[:, :1] * np.arange(K) + rng.standard_normal((n, K)), axis=1).astype(np.int32)
    return X, y


@pytest.mark.parametrize("rank", [B.RANK_FP32, B.RANK_EXACT], ids=["fp32", "exact"])
@pytest.mark.parametrize("n,p,K,trees,depth,mtry", [
    (2, 1, 2, 3, 4, 0), (3, 4, 2, 5, 3, 0), (65, 3, 3, 30, 9, 0), (600, 12, 4, 20, 11, 0),
    (300, 90, 2, 9, 8, 75), (900, 10, 6, 17, 10, 0), (700, 9, 13, 12, 12, 0),
    (260, 6, 3, 300, 6, 0), (4001, 5, 2, 11, 15, 0)])
def test_whole_trees_match_the_oracle_and_the_level_kernels(n, p, K, trees, depth, mtry, rank):
    X, y = problem(810 + n, n, p, K)
    kw = dict(max_iter=3, seed=5 + n, n_bins=64, mtry=mtry)
    print(f"whole trees n={n} p={p} K={K} T={trees} D={depth} mtry={mtry} rank={rank}", flush=True)
    o = O.boruta_fit(X, y, K, trees, depth, trace=True, **kw)
    for extra in (dict(), dict(graph=False), dict(tune=dict(col_level=64))):
        g = B.boruta_fit_ex(X, y, K, trees, depth, trace=True, split_rank=rank, **kw, **extra)
        assert_same_run(g, o)


def test_whole_trees_of_several_jobs():
    jobs = []
    for i, (n, p, K) in enumerate([(120, 5, 2), (700, 20, 3), (333, 8, 7)]):
        X, y = problem(830 + i, n, p, K)
        jobs.append(dict(X=X, y=y, n_classes=K, n_trees=8 + i, max_depth=6 + i, max_iter=4,
                         seed=60 + i, importance_mode=i % 2))
    batch = B.boruta_fit_batch(jobs, n_bins=64, trace=True)
    for j, jd in enumerate(jobs):
        o = O.boruta_fit(jd["X"], jd["y"], jd["n_classes"], jd["n_trees"], jd["max_depth"],
                         max_iter=4, seed=jd["seed"], importance_mode=jd["importance_mode"],
                         n_bins=64, trace=True)
        r = dict(batch["results"][j])
        r["traces"] = [t for t in batch["traces"] if t["job"] == j]
        assert_same_run(r, o)
