"""The selection of a band's trial frequencies where its bins can go wrong: every maximum taken, a few
of many, exact ties across the whole grid, more equal maxima than are sorted in LDS (the radix
select).  The n highest of a window are the first n of the 2n highest, and of all of them."""
import numpy as np
import pytest

from paper_1412_1840_amd import qmi

pytestmark = pytest.mark.gpu


def batch(kind, n, curves, rng):
    t = np.concatenate([np.sort(rng.uniform(0, 900, n)) if kind == "random"
                        else np.sort(rng.choice(1200, n, replace=False)).astype(float)
                        for _ in range(curves)])
    y = rng.normal(size=n * curves)
    return np.arange(curves + 1) * n, t, y, np.full(len(t), 0.1)


@pytest.mark.parametrize("kind,n,n_bands,n_grid", [
    ("random", 300, 6, 2), ("random", 300, 6, 700), ("random", 300, 6, 30000),
    ("integer", 300, 6, 641),  # periodic windows: 10 exact copies of every value
    ("integer", 300, 6, 64001),  # 1000 copies
    ("random", 20, 20, 30000),  # one sample per band: values that differ by rounding only
    ("integer", 20, 20, 64001),  # and not at all
])
def test_the_highest_are_a_prefix_of_more(kind, n, n_bands, n_grid):
    rng = np.random.default_rng(n_grid)
    off, t, y, e = batch(kind, n, 5, rng)
    f_hi = 1.0 / 64 + (n_grid - 1) / 64.0 if kind == "integer" else 10.0
    f_lo = 1.0 / 64 if kind == "integer" else 1e-3
    with qmi.Context(0) as ctx:
        def run(n_trials):
            _, trials, _ = ctx.bands_best_period(
                off, t, y, e, 0.3, f_lo=f_lo, f_hi=f_hi, n_bands=n_bands, n_keep=3,
                n_trials=n_trials, n_grid=n_grid)
            return np.asarray(trials).reshape(5, 3, n_trials)
        most = run(1024)
        found = np.isfinite(most).sum(2)
        for n_trials in (1, 2, 37, 150, 512, 1000):
            got = run(n_trials)
            assert np.array_equal(np.isfinite(got).sum(2), np.minimum(found, n_trials))
            np.testing.assert_array_equal(got, most[:, :, :n_trials])
