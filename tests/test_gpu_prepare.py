"""The preparation's LDS layout in batches (128 curves and more take the small block, whose sort needs
the least room): one, three, five and nine groups of harmonics, at lengths where the series tables,
not the sort keys, set the size in front of the operand tiles (an odd number of doubles for an odd
number of groups).  Values as in the mixed mode's other tests; the same bits alone, where the wide
block is used."""
import numpy as np
import pytest

import oracle as O
from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma_t,n", [(2.0, 40), (0.3, 121), (0.3, 256), (0.18, 200), (0.1, 300),
                                       (0.1, 512)])
def test_batches_of_short_curves(sigma_t, n):
    curves = [synth.survey_batch_curve(600 + k, n=n - k % 3) for k in range(130)]
    b = synth.pack(curves)
    f = np.concatenate([[0.0, 1.0], np.linspace(1e-3, 10.0, 30)])
    with qmi.Context(0) as ctx:
        sc, ips, ipy, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, f, sigma_t, want_ips=True)
        assert np.all(st == 0)
        for k in (0, 1, 2, 64, 129):
            c = curves[k]
            s1, i1, y1, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, f, sigma_t, want_ips=True)
            assert np.array_equal(s1[0], sc[k]) and np.array_equal(i1[0], ips[k]) and y1[0] == ipy[k]
            ref = O.information_potentials(c.t, c.y, sigma_t, O.silverman_sigma(c.y), f, mode=1)
            for i, v in enumerate((ref.vj, ref.ipt, ref.vc)):
                np.testing.assert_allclose(ips[k, :, i], v, rtol=2e-6)
