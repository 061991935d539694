"""A curve whose refined points all have one score (every sample at the same time): more equal points than
near ties are listed for.  The first point is taken, as the definition of the best says, and finding
that takes no longer than the search of an ordinary curve: at most 25 scans of the refined points, each
of which ends at the first few points that are too many, a microsecond or two."""
import time

import numpy as np
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("score", [qmi.SCORE_QMI, qmi.SCORE_NCKP])
def test_equal_times(score):
    n = 300
    c = synth.survey_batch_curve(970, n=n)
    kw = dict(f_min=1e-3, f_max=8.0, n_coarse=4000, top_k=10, n_fine=1000, score=score)
    with qmi.Context(0) as ctx:
        def run(t):
            best = np.inf
            for _ in range(10):
                t0 = time.perf_counter()
                res, coarse = ctx.best_period([0, n], t, c.y, c.e, 0.3, want_coarse=True, **kw)
                best = min(best, time.perf_counter() - t0)
            return res[0], coarse[0], best
        ordinary, _, t1 = run(c.t)
        for t in (np.full(n, 51234.5), np.zeros(n)):
            equal, coarse, t2 = run(t)
            assert equal["status"] == 0 and equal["reserved"] == 0
            assert np.abs(coarse).max() <= 1e-9 and np.all(coarse == coarse[0])
            assert abs(equal["score"]) <= 1e-9
            assert equal["coarse_argmax"] == 0
            assert t2 <= 1.5 * t1, (t1, t2)
