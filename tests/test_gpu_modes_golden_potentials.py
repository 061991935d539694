"""Potentials of the mixed mode against stored FP64 oracle values, at frequencies that include the
generating one of each periodic curve and its neighbours: there phases and magnitudes go together,
the node sums are largest and V_J takes their roundings in full.

Bound: the largest relative error of V_J, IP_t and V_C that the pair sums, with FP32 kernel values,
make on the same 16 curves x 256 frequencies (N = 1000): 2.9e-8, 8.7e-8 and 1.34e-8 for sigma_t 0.3,
0.1 and 0.6.  A sum over harmonics and nodes that stands in for them is to be no further off."""
import os

import numpy as np
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden",
                      "long_baseline_precision_oracle.npz")


@pytest.mark.parametrize("sigma_t,bound", [(0.3, 2.9e-8), (0.1, 8.7e-8), (0.6, 1.34e-8)])
def test_no_further_off_than_the_pair_sums(sigma_t, bound):
    g = np.load(GOLDEN)
    tag = "%g" % sigma_t
    worst = 0.0
    with qmi.Context(0) as ctx:
        for k, index in enumerate(g["k"]):
            c = synth.long_baseline_curve(int(index))
            _, ips, _, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, g["freqs"][k], sigma_t,
                                           want_ips=True)
            ref = np.stack([g[name + tag][k] for name in ("vj_", "ipt_", "vc_")], 1)
            worst = max(worst, np.abs(ips[0] / ref - 1).max())
    assert worst <= bound, worst
