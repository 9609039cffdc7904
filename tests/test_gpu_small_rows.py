"""The wave path's row limit: each chosen value is the one that acts, 32 among
them, from the caller and from a tuning cache; the library's choice is 64, less
in the plain form and for forests of many draws or few nodes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import autotune as A
from paper_2605_09950_amd import binding as B
from tests.parity_helpers import assert_same_run

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


def test_untouched_default_options_leave_the_choice_to_the_library():
    # the options of boruta_default_options hold 32: no choice unless another
    # launch parameter is set
    import ctypes
    rng = np.random.default_rng(61)
    X = rng.standard_normal((3000, 12)).astype(np.float32)
    y = np.argmax(X[:, :3] + rng.standard_normal((3000, 3)), axis=1).astype(np.int32)
    n = {}
    for unit in (2048, 0):
        o, st = B.boruta_default_options(), B.Stats()
        o.stats, o.col_unit = ctypes.pointer(st), unit
        out = [np.zeros(12, np.int8), np.zeros((2, 12)), np.zeros(1, np.int32)]
        ptr = [a.ctypes.data_as(ctypes.c_void_p) for a in (X, y, *out)]
        assert B.lib().boruta_fit_ex(ptr[0], ptr[1], 3000, 12, 3, 10, 10, 0, 0, 2, 0.05, 3,
                                     ctypes.byref(o), ptr[2], ptr[3], None, None, ptr[4]) == 0
        n[unit] = sum(st.level_small)
    assert n[2048] == wave_nodes(dict(small_rows=64))[0]
    assert n[0] == wave_nodes(dict(small_rows=32))[0]


def test_the_plain_form_keeps_to_32():
    n = {rows: wave_nodes(dict(small_rows=rows) if rows else None, form=B.FORM_PLAIN)[0]
         for rows in (0, 32, 64)}
    assert n[0] == n[32] < n[64]


@pytest.mark.parametrize("n,p,K,trees,depth,limit", [
    (300, 20, 0, 10, 8, 0), (600, 8, 0, 10, 8, 0), (200, 2200, 0, 20, 8, 0),  # no wave path
    (200, 600, 0, 60, 10, 32), (300, 8, 0, 10, 8, 64), (300, 20, 0, 400, 8, 64),
    (150, 2000, 2, 10, 6, 32), (150, 300, 3, 10, 6, 64)])
def test_the_limit_follows_the_forest(n, p, K, trees, depth, limit):
    # both sides of the rule's lines, regression (K = 0) and classification
    rng = np.random.default_rng(n + p)
    X = rng.standard_normal((n, p)).astype(np.float32)
    s = X[:, :3] + 0.5 * rng.standard_normal((n, 3))
    kw = dict(max_iter=2, seed=3, trace=True)
    print(f"library's limit n={n} p={p} K={K} T={trees} D={depth}: {limit}", flush=True)
    if K:
        y = np.argmax(s[:, :K], axis=1).astype(np.int32)
        o = O.boruta_fit(X, y, K, trees, depth, **kw)
        run = lambda **o: B.boruta_fit_ex(X, y, K, trees, depth, **kw, **o)  # noqa: E731
    else:
        y = s.sum(axis=1).astype(np.float32)
        o = O.boruta_fit_reg(X, y, trees, depth, **kw)
        run = lambda **o: B.boruta_fit_regression(X, y, trees, depth, **kw, **o)  # noqa: E731
    assert_same_run(run(), o)
    own = run(stats=True)
    assert_same_run(own, o)
    if limit:
        want = run(stats=True, tune=dict(small_rows=limit))
        other = run(stats=True, tune=dict(small_rows=96 - limit))
        assert list(own["stats"].level_small) == list(want["stats"].level_small)
        assert sum(own["stats"].level_small) != sum(other["stats"].level_small)
    else:
        assert sum(own["stats"].level_small) == 0
