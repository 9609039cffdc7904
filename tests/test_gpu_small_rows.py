"""The wave path's row limit: each chosen value is the one that acts, 32 among
them, from the caller and from a tuning cache; the library's choice is 64, and
32 in the plain form."""
import numpy as np
import pytest

from paper_2605_09950_amd import autotune as A
from paper_2605_09950_amd import binding as B

pytestmark = pytest.mark.gpu


def wave_nodes(tune=None, **kw):
    """Nodes that the wave path searched, and the run."""
    rng = np.random.default_rng(61)
    X = rng.standard_normal((3000, 12)).astype(np.float32)
    y = np.argmax(X[:, :3] + rng.standard_normal((3000, 3)), axis=1).astype(np.int32)
    r = B.boruta_fit_ex(X, y, 3, 10, 10, max_iter=2, seed=3, stats=True, tune=tune, **kw)
    return sum(r["stats"].level_small), r


def test_every_chosen_limit_acts(tmp_path):
    runs = {rows: wave_nodes(dict(small_rows=rows)) for rows in (31, 32, 33, 64)}
    n = {rows: runs[rows][0] for rows in runs}
    print(f"wave-path nodes by limit: {n}", flush=True)
    assert n[31] <= n[32] <= n[33] < n[64]
    none, base = wave_nodes()
    assert none == n[64]
    cache = str(tmp_path / "tune.txt")
    jd = dict(X=np.zeros((3000, 12), np.float32), n_classes=3, n_trees=10, max_depth=10)
    A.write_cache(cache, {A.signature([jd]): dict(small_rows=32)})
    assert wave_nodes(dict(tune_cache=cache))[0] == n[32]
    for _, r in runs.values():
        for k in ("decision", "hits", "shadow_max", "imp_history"):
            assert np.array_equal(r[k], base[k], equal_nan=True)


def test_the_plain_form_keeps_to_32():
    n = {rows: wave_nodes(dict(small_rows=rows) if rows else None, form=B.FORM_PLAIN)[0]
         for rows in (0, 32, 64)}
    assert n[0] == n[32] < n[64]
