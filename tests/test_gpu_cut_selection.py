"""Columns longer than a sort tile take their cuts by selection: bins against the
oracle's at the first such length and ragged ones, two to 256 bins, and columns
whose keys share digits: few values, one value, one-ulp steps, both signs and zeros,
huge and tiny magnitudes.  Bytes: no tolerance."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_09950_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_bins", [(8192, 256), (8193, 256), (8193, 2), (16386, 17),
                                      (20003, 256), (131073, 255)])
def test_selected_cuts_give_the_oracle_bins(n, n_bins):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 9)).astype(np.float32)
    X[:, 1] = rng.integers(0, 2, n)
    X[:, 2] = -3.25
    X[:, 3] = (np.float32(1.0).view(np.int32) + rng.integers(0, 900, n)).astype(
        np.int32).view(np.float32)
    X[:, 4] = np.where(rng.random(n) < 0.7, -0.0, X[:, 4])
    X[:, 5] = np.exp(40 * X[:, 5].clip(-2, 2)) * np.sign(X[:, 0])
    X[:, 6] = np.sort(X[:, 6])
    X[:, 7] = np.arange(n)[::-1] // 3
    X[:, 8] = np.where(np.arange(n) == n - 1, 3e38, -3e38)
    print(f"cuts n={n} bins={n_bins}", flush=True)
    want, _, _ = O.bin_matrix(X, n_bins)
    assert np.array_equal(B.boruta_bin(X, n_bins), want)
