"""Class counts packed in 8- and 16-bit fields (nodes below a weight of 256 and
of 65536) against the oracle, at the places where the forms and the scans
change: nodes of 1 to 64, 65 to 128 and more rows, weights around 256, 2 to 16
classes, columns of few distinct values (many thresholds tie exactly, mirrored
partitions among them), both histogram layouts, both ranking modes.  All
results are integers or quotients of integers: the tolerance is zero."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

pytestmark = pytest.mark.gpu


def problem(seed, n, p, K, levels):
    rng = np.random.default_rng(seed)
    X = rng.integers(0, levels, (n, p)).astype(np.float32)
    s = X[:, :1] * np.arange(1, K + 1) / levels + rng.standard_normal((n, K))
    return X, np.argmax(s, axis=1).astype(np.int32)


def same(K, n, trees, depth, iters, tune, rank, levels=9, p=7):
    X, y = problem(500 + 10 * K + n % 7, n, p, K, levels)
    kw = dict(max_iter=iters, seed=31 + K, n_bins=64)
    print(f"packed counts K={K} n={n} levels={levels} tune={tune} rank={rank}", flush=True)
    g = B.boruta_fit_ex(X, y, K, trees, depth, trace=True, tune=tune, split_rank=rank, **kw)
    o = O.boruta_fit(X, y, K, trees, depth, trace=True, **kw)
    assert_same_run(g, o)


@pytest.mark.parametrize("rank", [B.RANK_FP32, B.RANK_EXACT], ids=["fp32", "exact"])
@pytest.mark.parametrize("tune", [dict(small_rows=2, col_level=64), dict(small_rows=2, col_level=1),
                                  dict(small_rows=64)], ids=["node_major", "column", "wave64"])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 8, 9, 16])
def test_tied_thresholds_at_every_node_size(K, tune, rank):
    # small_rows = 2: nodes of 3 to 190 rows all take the histogram path
    same(K, 300, 40, 10, 2, tune, rank)


@pytest.mark.parametrize("col", [64, 1], ids=["node_major", "column"])
@pytest.mark.parametrize("K", [2, 3, 4, 6, 11])
def test_weights_around_the_eight_bit_limit(K, col):
    # roots of about 160 rows and a weight of 255, 256 and 257; 1.6 times these below
    for n in (255, 256, 257, 420):
        same(K, n, 12, 4, 2, dict(col_level=col), B.RANK_FP32, levels=50)


@pytest.mark.parametrize("K", [2, 3, 4, 7, 12])
@pytest.mark.parametrize("n", [65535, 65536])
def test_weights_around_the_sixteen_bit_limit(n, K):
    same(K, n, 2, 3, 1, dict(col_level=1 if K in (4, 12) else 64), B.RANK_FP32, levels=60, p=3)


@pytest.mark.parametrize("rank", [B.RANK_FP32, B.RANK_EXACT], ids=["fp64", "exact"])
@pytest.mark.parametrize("rows", [2, 7, 16, 32, 64])
@pytest.mark.parametrize("kind", ["ties", "wide"])
def test_regression_nodes_of_the_wave_path(kind, rows, rank):
    # target sums as FP64 integers in nodes of up to 64 rows: tied thresholds
    # (few targets and bin values), targets over many binades, both rankings
    rng = np.random.default_rng(640 + rows)
    X = rng.integers(0, 12, (400, 9)).astype(np.float32)
    y = np.round(X[:, 0] - X[:, 1] + rng.standard_normal(400))
    if kind == "wide":
        y = (y - 3) * np.exp(rng.uniform(-30, 0, 400))
    kw = dict(max_iter=3, seed=9 + rows, n_bins=64)
    print(f"regression wave path rows={rows} kind={kind} rank={rank}", flush=True)
    g = B.boruta_fit_regression(X, y.astype(np.float32), 30, 12, trace=True, split_rank=rank,
                                tune=dict(small_rows=rows), **kw)
    o = O.boruta_fit_reg(X, y.astype(np.float32), 30, 12, trace=True, **kw)
    assert_same_run(g, o)
