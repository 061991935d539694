"""The mode sums in FP64 against the pair sums, written out, where their layout can go wrong: lengths around the
block of four samples and around the length from which they are used, one harmonic group and many,
magnitudes in few or many node quads, so scattered that the pair sums take the curve over, both launch
forms.

Tolerances: the phase of harmonic m carries m rounding errors of 6e-17 turns (at most 100 here: 4e-14
of a value, independent from sample to sample), sums of up to 2049 samples as many of 1e-16, and the
node sums are off by at most 8e-14 of a kernel value (all samples at the same place between two
nodes): V's are held to 1e-12, and QMI, the sum of four logarithms of such values, to 4e-12."""
import numpy as np
import pytest

import oracle as O
from paper_1412_1840_amd import qmi, synth
from test_gpu_modes import clumped

pytestmark = pytest.mark.gpu

V_RTOL, QMI_ABS = 1e-12, 4e-12
FREQS = np.concatenate([[0.0, 1.0], np.linspace(1e-3, 10.0, 33), [1 / 3.7]])


@pytest.fixture(scope="module")
def ctx():
    with qmi.Context(0) as c:
        yield c


def potentials(c, st, sy):
    """V_J, IP_t, V_C at FREQS and IP_y.  Phases are folded in extended precision: f (t_i - t_j) in
    double is off by up to 4e-12 turns here, which the oracle's potentials show at sigma_t = 0.1."""
    A, B = (1 / np.sqrt(2 * np.pi) / w for w in (st, sy))
    K = B * np.exp(-((c.y[:, None] - c.y[None, :]) / sy) ** 2 / 2)
    r = K.sum(1)
    out = np.empty((len(FREQS), 3))
    for k, f in enumerate(FREQS):
        p = np.longdouble(f) * c.t.astype(np.longdouble)
        p -= np.rint(p)
        d = (p[:, None] - p[None, :]).astype(np.float64)
        g = A * np.exp(-2 * np.sin(np.pi * d) ** 2 / st ** 2)
        out[k] = (K * g).sum() / c.n ** 2, g.sum() / c.n ** 2, r @ g.sum(1) / c.n ** 3
    return out, r.sum() / c.n ** 2


def check(c, sc, ips, ipy, st, sy):
    v, vy = potentials(c, st, sy)
    np.testing.assert_allclose(ips, v, rtol=V_RTOL, err_msg="n=%d" % c.n)
    np.testing.assert_allclose(ipy, vy, rtol=V_RTOL)
    err = np.abs(sc - (np.log(v[:, 0]) + np.log(vy * v[:, 1]) - 2 * np.log(v[:, 2])))
    assert err.max() <= QMI_ABS and abs(sc[0]) <= 1e-14, (c.n, err.max(), sc[0])


@pytest.mark.parametrize("sigma_t,lengths", [
    (0.3, [187, 188, 189, 190, 191, 192, 193, 256, 257, 617, 2049]),  # 9 groups
    (0.6, [100, 101, 102, 103, 104, 128, 300]),
    (2.0, [59, 60, 61, 62, 63, 64, 65]),
    (9.0, [40, 41, 43, 44]),  # one group
    (0.1, [511, 512, 513, 514, 700]),
])
def test_lengths_and_groups(ctx, sigma_t, lengths):
    curves = [synth.survey_batch_curve(700 + k, n=n) for k, n in enumerate(lengths)]
    b = synth.pack(curves)
    sc, ips, ipy, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, FREQS, sigma_t, want_ips=True,
                                       precision=qmi.PREC_FP64)
    assert np.all(st == 0)
    for k, c in enumerate(curves):
        check(c, sc[k], ips[k], ipy[k], sigma_t, O.silverman_sigma(c.y))


@pytest.mark.parametrize("kind", ["line", "pairs", "two", "steps", "tail"])
def test_magnitude_distributions(ctx, kind):
    rng = np.random.default_rng(6)
    for n in (190, 503):
        c = clumped(kind, n, rng)
        for sy in (50.0, 0.7, 0.11, 0.02, 1e-3, 1e-7):
            sc, ips, ipy, st = ctx.periodogram([0, n], c.t, c.y, c.e, FREQS, 0.3, sigma_y=sy,
                                               want_ips=True, precision=qmi.PREC_FP64)
            assert st[0] == 0
            check(c, sc[0], ips[0], ipy[0], 0.3, sy)


def test_longest_curve_against_the_mixed_sums(ctx):
    c = synth.survey_batch_curve(9, n=qmi.MAX_N)
    a, b = (ctx.periodogram([0, c.n], c.t, c.y, c.e, FREQS, 0.3, want_ips=True, precision=p)
            for p in (qmi.PREC_FP64, qmi.PREC_MIXED))
    assert abs(a[0][0, 0]) <= 1e-14
    np.testing.assert_allclose(a[1], b[1], rtol=2e-6)  # the mixed sums' own tolerance


def test_both_launch_forms_and_given_back_curves(ctx):
    """33 curves of 4096 frequencies run every group in one wave, each alone a group per wave: the
    same bits.  Scattered curves among them go to the pair sums, from host and device arrays,
    without allocation, and in a search, as they do alone."""
    rng = np.random.default_rng(8)
    curves = [synth.survey_batch_curve(800 + k, n=190 + 3 * k) for k in range(33)]
    for k in (0, 7, 8, 32):
        curves[k] = clumped("tail", curves[k].n, rng)
    b = synth.pack(curves)
    f = np.linspace(0.0, 10.0, 4096)
    kw = dict(sigma_y=1e-3, precision=qmi.PREC_FP64)
    sc, ips, ipy, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, f, 0.3, want_ips=True, **kw)
    assert np.all(st == 0)
    few = dict(f_min=1e-3, f_max=3.0, n_coarse=1500, top_k=3, n_fine=40)
    res, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **few, **kw)
    import torch
    for k in (0, 1, 7, 8, 20, 32):
        c = curves[k]
        s1, i1, y1, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, f, 0.3, want_ips=True, **kw)
        assert np.array_equal(s1[0], sc[k]) and np.array_equal(i1[0], ips[k]) and y1[0] == ipy[k]
        r1, _ = ctx.best_period([0, c.n], c.t, c.y, c.e, 0.3, **few, **kw)
        for name in ("f_best", "score", "score_nckp", "fine_index"):
            assert r1[name][0] == res[name][k], (k, name)
        dev = [torch.from_numpy(a).cuda() for a in (c.t, c.y, c.e, f[:50])]
        out = torch.empty((1, 50), dtype=torch.float64, device="cuda")
        ctx.periodogram_noalloc([0, c.n], *dev, out, 0.3, **kw)
        assert np.array_equal(out.cpu().numpy()[0], sc[k][:50])
