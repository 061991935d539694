"""The register sorts of the preparation kernels at the lengths where their layout changes: below
and above 256, 512, 1024, 2048, 4096 keys and at the longest, with ties, through entry points whose
results show the order: whitening (stable phase order, bitwise against the oracle) and the kernel
widths and pSNR (order statistics; rounding of the mean and of 0.9 ... N^-0.2 only)."""
import numpy as np
import pytest

import oracle as O
from paper_1412_1840_amd import qmi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 130])  # a few curves (wide blocks), and a batch
@pytest.mark.parametrize("n", [2, 63, 64, 65, 255, 256, 257, 512, 513, 1023, 1024, 1025, 2048, 2049,
                               4097, 8191, 8192])
def test_orders(n, copies):
    if copies > 1 and n > 1100:
        pytest.skip("one block shape above 1024 samples")
    rng = np.random.default_rng(n)
    t = np.round(rng.uniform(0, 300, n), 1)  # many equal phases
    y = np.round(rng.normal(size=n), 2)
    e = np.round(rng.uniform(0.1, 0.3, n), 2)
    off = np.arange(copies + 1) * n
    T, Y, E = (np.tile(a, copies) for a in (t, y, e))
    with qmi.Context(0) as ctx:
        yw, st = ctx.whiten(off, T, Y, np.full(copies, 2.5), window=7)
        assert np.all(st == 0)
        ref = O.whiten(t, y, 2.5, 7)
        res, _ = ctx.best_period(off, T, Y, E, 0.3, 0.1, 0.2, 2, top_k=0, n_fine=0)
    for k in range(copies):
        assert np.array_equal(yw[k * n:(k + 1) * n], ref), k
        assert res["psnr"][k] == pytest.approx(O.psnr(y, e), rel=1e-14)
        assert res["sigma_y"][k] == pytest.approx(O.silverman_sigma(y), rel=1e-12)
