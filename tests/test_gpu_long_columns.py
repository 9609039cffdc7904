"""Bins of very long columns: few of them are sorted by the whole chip, more take
their cuts by selection; both sides of both lines against the oracle.  Bytes: no
tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,n_bins", [(1 << 18, 3, 256), ((1 << 18) + 1, 1, 256),
                                        ((1 << 18) + 1, 8, 100), ((1 << 18) + 1, 9, 100),
                                        (524289, 4, 255), (1 << 19, 2, 2), (786433, 16, 33)])
def test_bins_of_long_columns_match_the_oracle(n, p, n_bins):
    rng = np.random.default_rng(n + p)
    X = rng.standard_normal((n, p)).astype(np.float32)
    X[:, 0] = np.where(rng.random(n) < 0.7, -0.0, X[:, 0])
    if p > 2:
        X[:, 1] = rng.integers(0, 5, n)
        X[:, 2] = np.where(np.arange(n) == n - 1, 3e38, -3e38)
    print(f"long columns n={n} p={p} bins={n_bins}", flush=True)
    want, _, _ = O.bin_matrix(X, n_bins)
    assert np.array_equal(B.boruta_bin(X, n_bins), want)
