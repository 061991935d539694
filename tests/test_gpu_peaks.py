"""The scan for the highest local maxima where its split can go wrong: grids around the length of a
part, one part and the most, lists shorter than top_k, ties.  The records are compared with the
maxima that numpy finds in the periodogram that the search itself returns (exactly: the scan only
compares), and a curve's record alone (a split scan) with its record in a batch (an unsplit one)."""
import numpy as np
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


def maxima(q, top_k):
    """Grid indices of the top_k local maxima by (score descending, index ascending)."""
    left = np.concatenate([[True], q[1:] > q[:-1]])
    right = np.concatenate([q[:-1] >= q[1:], [True]])
    k = np.nonzero(left & right)[0]
    return k[np.lexsort((k, -q[k]))][:top_k]


@pytest.mark.parametrize("top_k", [1, 10, 32])
@pytest.mark.parametrize("n_coarse", [1, 2, 30, 1023, 1024, 2047, 2048, 2049, 5000, 20001, 40000])
def test_maxima_of_split_and_unsplit_scans(n_coarse, top_k):
    curves = [synth.survey_batch_curve(40 + k, n=60 + k) for k in range(4)]
    flat = synth.Curve(np.arange(64.0), np.tile([0.0, 1.0], 32), np.full(64, 0.1), False)
    curves.append(flat)  # sampled once a day: the periodogram repeats with period 1, exact ties
    b = synth.pack(curves * 60)
    kw = dict(f_min=0.0, f_max=4.0, n_coarse=n_coarse, top_k=top_k, n_fine=1000)
    with qmi.Context(0) as ctx:
        many, coarse = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, want_coarse=True, **kw)
        for k, c in enumerate(curves):
            one, q = ctx.best_period([0, c.n], c.t, c.y, c.e, 0.3, want_coarse=True, **kw)
            np.testing.assert_array_equal(q[0], coarse[k])
            want = maxima(q[0], top_k)
            for r in (one[0], many[k], many[k + len(curves)]):
                assert r["n_peaks"] == len(want)
                assert r["coarse_argmax"] == np.argmax(q[0])
                assert r["coarse_best"] == q[0].max()
                assert r["coarse_index"] == want[r["peak_rank"]]
            for name in ("f_best", "score", "peak_rank", "fine_index"):
                assert one[0][name] == many[k][name]
