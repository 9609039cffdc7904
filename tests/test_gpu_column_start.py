"""Where the column-major levels of a matrix past 128 MiB start: at level 3 when a
column has enough items there, else at 5; the results are those of node-major
levels throughout, whatever the start."""
import numpy as np
import pytest

from paper_2605_09950_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trees,depth,mtry,levels", [(4, 7, 0, 2), (4, 5, 0, 0), (200, 4, 5000, 1)],
                         ids=["few", "few_shallow", "many"])
def test_column_levels_start_by_the_items_per_column(trees, depth, mtry, levels):
    rng = np.random.default_rng(88)
    X = rng.standard_normal((260, 140000), dtype=np.float32)  # widened: 280,000 columns of 512 bytes
    y = (X[:, 0] + X[:, 1] + 0.5 * rng.standard_normal(260) > 0).astype(np.int32)
    kw = dict(max_iter=1, seed=2, n_bins=64, mtry=mtry)
    print(f"column start T={trees} D={depth} mtry={mtry}: {levels} levels", flush=True)
    a = B.boruta_fit_ex(X, y, 2, trees, depth, stats=True, **kw)
    assert a["stats"].hist_col.launches == levels
    b = B.boruta_fit_ex(X, y, 2, trees, depth, tune=dict(col_level=64), **kw)
    for k in ("decision", "hits", "imp_history", "shadow_max"):
        assert np.array_equal(a[k], b[k], equal_nan=True)
