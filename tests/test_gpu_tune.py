"""The variant probe of the pair sums and the pass that decides near ties share the pair sums'
buffers.  A fresh context's first call both tunes (more than 2e9 pair x frequency items on curves of
the pair sums) and decides ties of longer curves, whose tables are larger than the group's own: the
probe has to be over by then.  The records are those of each curve alone, on contexts of their own,
which tune nothing or decide their ties with no other curve beside them."""
import numpy as np
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma_t", [0.1, qmi.SIGMA_T_SKEWNESS])
def test_first_call_tunes_and_decides_ties(sigma_t):
    curves = [synth.survey_batch_curve(900 + k, n=n)
              for k, n in enumerate([250, 251, 260, 270, 1000, 900, 1100, 700])]
    b = synth.pack(curves)
    # windows of 20 000 points: every curve of the mode sums has near ties (1e-8 of the score)
    kw = dict(f_min=1e-3, f_max=10.0, n_coarse=30000, top_k=2, n_fine=20000)
    assert sum(0.5 * c.n * (c.n - 1) * kw["n_coarse"] for c in curves[:4]) > 2e9
    with qmi.Context(0) as ctx:
        first, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, sigma_t, **kw)
        again, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, sigma_t, **kw)
        assert first.tobytes() == again.tobytes()
        assert np.all(first["status"] == 0) and np.all(first["reserved"] == 0)
        for k, c in enumerate(curves):
            one, _ = ctx.best_period([0, c.n], c.t, c.y, c.e, sigma_t, **kw)
            assert one.tobytes() == first[k:k + 1].tobytes(), k
