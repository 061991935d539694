"""qmi_preprocess writes offsets and statuses only once every sample is down: the new offsets may
then take the place of the batch's own, and of its samples (the copies are exact)."""
import ctypes

import numpy as np
import pytest

from paper_1412_1840_amd import qmi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_curves", [1, 7, 300])
def test_outputs_in_place_of_the_inputs(n_curves):
    rng = np.random.default_rng(n_curves)
    lens = rng.integers(1, 400, n_curves)  # those below 50 samples are rejected
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    t, y = rng.uniform(0, 900, off[-1]), rng.normal(0, 1, off[-1])
    e = rng.lognormal(-2.5, 0.7, off[-1])
    with qmi.Context(0) as ctx:
        oo, to, yo, eo, st, det = ctx.preprocess(off, t, y, e)
        st2, det2 = np.zeros(n_curves, np.int32), np.zeros(n_curves, np.uint8)
        b, off2 = ctx._batch(off.copy(), t, y, e)
        pp = qmi.PreprocessParams(1, 50, 1, 0)
        ctx._check(qmi.lib().qmi_preprocess(
            ctx._h, ctypes.byref(b), ctypes.byref(pp), off2.ctypes.data, t.ctypes.data,
            y.ctypes.data, e.ctypes.data, st2.ctypes.data, det2.ctypes.data))
    m = int(oo[-1])
    assert np.array_equal(off2, oo) and np.array_equal(st2, st) and np.array_equal(det2, det)
    assert np.array_equal(t[:m], to) and np.array_equal(y[:m], yo) and np.array_equal(e[:m], eo)
