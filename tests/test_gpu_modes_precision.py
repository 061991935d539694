"""Errors of the mixed mode's potentials where the mode sums could lose some: long sums (8192 samples,
wide magnitude kernels that put every sample in one group), phases that coincide or nearly do, and
times on a grid at multiples of its frequency.

Tolerance of the rms relative error over the frequencies.  A value of a harmonic carries about six
independent roundings of 1.7e-8 rms (two parts of 11 bits, sine, cosine, recurrence): 4e-8, which
enters |a|^2 twice and averages over N samples: 8e-8 / sqrt(N), at worst with all phases alike.  A
node's sum is rounded once per block of 32 samples, 2.6e-8 rms of what was summed since the last of
the 8-block carries, at most 8 such sums of growing size: 2.6e-8 sqrt(8 / 3), averaged over some 30
nodes and entering twice: 1.5e-8 / sqrt(30) x 2 = 1.5e-8 / 2.7 = 5.5e-9 at worst.  Both together,
with half as much again for the spread from curve to curve: 1.2e-7 / sqrt(N) + 8e-9.
At f = 0 the potentials are exact up to the nodes: V_J - V_M is 2e-9 of V_J at most (the pair sums:
exactly 0)."""
import numpy as np
import pytest

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with qmi.Context(0) as c:
        yield c


def errors(ctx, t, y, freqs, sigma_t, sigma_y):
    e = np.full(len(t), 0.1)
    kw = dict(want_ips=True, sigma_y=sigma_y)
    got, ref = (ctx.periodogram([0, len(t)], t, y, e, freqs, sigma_t, precision=p, **kw)[1][0]
                for p in (qmi.PREC_MIXED, qmi.PREC_FP64))
    return got, got / ref - 1


RNG = np.random.default_rng(3)
COHERENT = np.concatenate([RNG.uniform(1e-4, 3e-3, 60), 1 + RNG.uniform(-1e-3, 1e-3, 60)])
SPREAD = RNG.uniform(1e-3, 10.0, 120)


@pytest.mark.parametrize("freqs", [COHERENT, SPREAD], ids=["coherent", "spread"])
@pytest.mark.parametrize("n,sigma_t,sigma_y", [
    (121, 0.3, -1.0), (121, 0.6, -1.0), (330, 0.3, -1.0), (617, 0.3, -1.0), (617, 0.1, -1.0),
    (1000, 0.6, -1.0), (2500, 0.3, -1.0), (8192, 0.3, -1.0), (617, 0.3, 50.0), (8192, 0.3, 50.0),
    (8192, 0.6, 1.0)])
def test_errors_of_the_potentials(ctx, freqs, n, sigma_t, sigma_y):
    c = synth.survey_batch_curve(40, n=n)
    _, rel = errors(ctx, c.t, c.y, freqs, sigma_t, sigma_y)
    rms = np.sqrt((rel ** 2).mean(0))
    assert rms.max() <= 1.2e-7 / np.sqrt(n) + 8e-9, rms


@pytest.mark.parametrize("sigma_t", [0.04, 0.1, 0.3, 0.6])
@pytest.mark.parametrize("n", [200, 700])
def test_times_on_a_grid(ctx, n, sigma_t):
    """Four samples a day: all phases coincide at multiples of 4, and take two, four, ... values at
    the fractions (a few values of sine and cosine, whose roundings do not average out: 3e-8 and
    less each, twice, for the pair sums as for the mode sums)."""
    rng = np.random.default_rng(n)
    t = np.sort(rng.choice(4 * n, n, replace=False)) * 0.25
    y = synth.survey_batch_curve(41, n=n).y
    freqs = np.array([0.0, 4.0, 8.0, 0.25, 0.5, 1.0, 1.5, 2.0, 3.0, 5.0])
    got, rel = errors(ctx, t, y, freqs, sigma_t, -1.0)
    assert np.abs(rel).max() <= 6e-8, rel
    assert np.sqrt((rel ** 2).mean(0)).max() <= 3e-8


def test_zero_frequency(ctx):
    for n in (150, 617, 4000):
        c = synth.survey_batch_curve(42, n=n)
        _, ips, ipy, _ = ctx.periodogram([0, n], c.t, c.y, c.e, np.array([0.0, 0.1]), 0.3,
                                         want_ips=True)
        vj, ipt, _ = ips[0, 0]
        assert abs(vj - ipy[0] * ipt) <= 2e-9 * vj


@pytest.mark.parametrize("precision", [qmi.PREC_MIXED, qmi.PREC_FP64])
def test_all_phases_alike(ctx, precision):
    """Equal times at any frequency, and times on a grid at multiples of its frequency: the kernel of
    times is 1 everywhere, so that V_J = V_M = V_C up to the rounding of the FP64 steps that follow, 1e-15
    of nCKP's scale sqrt(N st) IP_t / IP_y = sqrt(N / st) / sqrt(2 pi) and a dozen of them."""
    for n in (300, 617, 3000):
        y = synth.survey_batch_curve(43, n=n).y
        e = np.full(n, 0.1)
        for t, f in ((np.full(n, 51234.5678), [0.0, 1e-3, 0.37, 9.1]),
                     (50000 + 0.25 * np.arange(n), [4.0, 8.0, 400.0])):
            kw = dict(precision=precision)
            q, _, _, _ = ctx.periodogram([0, n], t, y, e, np.array(f), 0.3, **kw)
            c, _, _, _ = ctx.periodogram([0, n], t, y, e, np.array(f), 0.3, score=qmi.SCORE_NCKP, **kw)
            assert np.abs(q).max() <= 1e-13 and np.abs(c).max() <= 1e-13 * np.sqrt(n / 0.3)
