"""Errors of the FP64 mode sums where their nodes could show: magnitudes that all lie at the same place
between two nodes (a wide kernel, a few values, steps of the magnitudes that are whole node spacings),
one magnitude far from the others, and lengths around the one from which the sums are used and around
the blocks of four samples.

Tolerances: the phase of harmonic m (33 at sigma_t 0.3, 19 at 0.6) carries m roundings of 6e-17 turns,
4e-16 of a value times m at worst, independent over the samples: 2 x 1.2e-14 / sqrt(N) of a sum, 2e-15
at 150 samples; the trapezoid rule 6e-17; sums of up to 1000 terms as many roundings of 1e-16, here
and in the reference, of which some 30 remain: 3e-15.  V's are held to 1e-14, QMI, the sum of four
logarithms, to 3e-14."""
import numpy as np
import pytest

import oracle as O
from paper_1412_1840_amd import qmi, synth
from test_gpu_modes64 import FREQS, potentials

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with qmi.Context(0) as c:
        yield c


def check(ctx, c, sigma_t, sigma_y):
    sc, ips, ipy, st = ctx.periodogram([0, c.n], c.t, c.y, c.e, FREQS, sigma_t, sigma_y=sigma_y,
                                       want_ips=True, precision=qmi.PREC_FP64)
    assert st[0] == 0
    v, vy = potentials(c, sigma_t, sigma_y)
    np.testing.assert_allclose(ips[0], v, rtol=1e-14)
    np.testing.assert_allclose(ipy[0], vy, rtol=1e-14)
    q = np.log(v[:, 0]) + np.log(vy * v[:, 1]) - 2 * np.log(v[:, 2])
    assert np.abs(sc[0] - q).max() <= 3e-14


def curve(n, y):
    return synth.Curve(synth.survey_batch_curve(60, n=n).t, np.asarray(y, dtype=float),
                       np.full(n, 0.1), False)


@pytest.mark.parametrize("n", [250, 617])
@pytest.mark.parametrize("sigma_y", [50.0, 3.0])
def test_kernels_wider_than_the_magnitudes(ctx, n, sigma_y):
    check(ctx, synth.survey_batch_curve(61, n=n), 0.3, sigma_y)


@pytest.mark.parametrize("step", [0.36, 0.4, 0.72, 0.9, 0.18])
def test_magnitudes_in_steps(ctx, step):
    rng = np.random.default_rng(4)
    y = 15.0 + 0.02 * step * rng.integers(0, 12, 300)  # in units of sigma_y
    check(ctx, curve(300, y), 0.3, 0.02)


def test_equal_magnitudes(ctx):
    check(ctx, curve(300, np.full(300, 17.25)), 0.3, 0.05)


@pytest.mark.parametrize("far", [-9999.0, 99.999, 1e6])
def test_one_magnitude_far_from_the_others(ctx, far):
    y = synth.survey_batch_curve(62, n=400).y.copy()
    y[123] = far
    check(ctx, curve(400, y), 0.3, 0.05)


@pytest.mark.parametrize("sigma_t,lengths", [
    (2.0, [69, 70, 71, 72, 73]), (0.6, [144, 145, 146, 147, 148]),
    (0.3, [244, 245, 246, 247, 248]), (0.1, [694, 695, 697])])
def test_lengths(ctx, sigma_t, lengths):
    for n in lengths:
        c = synth.survey_batch_curve(63, n=n)
        check(ctx, c, sigma_t, O.silverman_sigma(c.y))
