"""Near ties are decided by the pair sums under any memory budget that a call accepts: where the
budget has just room for the group's own buffers, the tables for the ties take the place of others
and the tied curves are scored a few at a time.  Every budget gives the records of a large one."""
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


def test_every_budget_gives_the_same_records():
    # windows of 20 000 points on flat maxima: every curve has near ties (1e-8 of the score)
    curves = [synth.survey_batch_curve(950 + k, n=400 - k % 5) for k in range(40)]
    b = synth.pack(curves)
    kw = dict(f_min=1e-3, f_max=2.0, n_coarse=2500, top_k=3, n_fine=20000)
    with qmi.Context(0) as ctx:
        ref, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
    ran = 0
    for mb in (3, 4, 6, 9, 13, 20, 30, 45, 60, 70, 80, 85, 90, 95, 100, 105, 110, 120, 140):
        with qmi.Context(0, budget_bytes=mb << 20) as ctx:
            try:
                res, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
            except qmi.QMIError as e:  # not even one curve fits
                assert e.code == qmi.ENOMEM and mb < 6
                continue
            again, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
        ran += 1
        assert res.tobytes() == ref.tobytes(), mb
        assert again.tobytes() == ref.tobytes(), mb
    assert ran >= 15
