"""The mode sums (harmonics x magnitude nodes) against the FP64 oracle where their layout can go
wrong: lengths around the block of 32 samples and around the length from which they are used, one
harmonic group and several, magnitudes that fill few or many node blocks, so scattered that the
pair sums take the curve over (alone and between others, through every entry point), and both
launch forms.

Tolerances: a value of the operands is rounded to half precision twice, 2^-24 of its size, and a
harmonic is at most six recurrence steps from its hardware sine and cosine (measured error 6e-7
rms), each sample independently; a sum over at least 40 samples and several harmonics averages
these to below 3e-7 of V_J, IP_t and V_C, and FP32 accumulation adds at most 3 x blocks roundings,
random in sign, of 6e-8.  V's are held to 2e-6 and QMI to 1e-4 as everywhere in the mixed mode, and
QMI to 2e-6 absolute here: the errors of the V's cancel in it to first order."""
import numpy as np
import pytest

import oracle as O
from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu

V_RTOL, QMI_TOL, QMI_ABS = 2e-6, 1e-4, 2e-6
FREQS = np.concatenate([[0.0, 1.0], np.linspace(1e-3, 10.0, 37), [1 / 3.7]])


@pytest.fixture(scope="module")
def ctx():
    with qmi.Context(0) as c:
        yield c


def check(c, sc, ips, st, sy):
    ref = O.information_potentials(c.t, c.y, st, sy, FREQS, mode=1)
    q = O.qmi(ref)
    for i, v in enumerate((ref.vj, ref.ipt, ref.vc)):
        np.testing.assert_allclose(ips[:, i], v, rtol=V_RTOL, err_msg="n=%d V %d" % (c.n, i))
    err = np.abs(sc - q)
    assert np.all(err <= QMI_TOL * np.maximum(np.abs(q), 1e-3 * np.max(np.abs(q)))), (c.n, err.max())
    assert err.max() <= QMI_ABS and abs(sc[0]) <= 1e-12, (c.n, err.max(), sc[0])


@pytest.mark.parametrize("sigma_t,lengths", [
    (0.3, [79, 95, 96, 97, 127, 128, 129, 160, 161, 511, 2049]),  # 3 groups
    (0.6, [39, 47, 48, 63, 64, 65, 96, 257]),  # 2 groups
    (2.0, [24, 31, 32, 33, 64, 100]),  # 1 group
    (0.1, [255, 288, 289, 320, 353, 700]),  # 9 groups
    (0.04, [600, 700, 1024]),
])
def test_lengths_and_groups(ctx, sigma_t, lengths):
    curves = [synth.survey_batch_curve(300 + k, n=n) for k, n in enumerate(lengths)]
    b = synth.pack(curves)
    sc, ips, _, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, FREQS, sigma_t, want_ips=True)
    assert np.all(st == 0)
    for k, c in enumerate(curves):
        check(c, sc[k], ips[k], sigma_t, O.silverman_sigma(c.y))


def clumped(kind, n, rng):
    y = {"line": rng.uniform(0, 1, n), "pairs": np.repeat(np.arange(n // 2 + 1), 2)[:n] * 1.0,
         "two": np.where(np.arange(n) % 3 == 0, 5.0, 0.0) + 1e-3 * rng.normal(size=n),
         "steps": np.floor(rng.uniform(0, 6, n)), "tail": np.exp(3 * rng.normal(size=n))}[kind]
    return synth.Curve(np.sort(rng.uniform(0, 900, n)), y[rng.permutation(n)], np.full(n, 0.1), False)


@pytest.mark.parametrize("kind", ["line", "pairs", "two", "steps", "tail"])
def test_magnitude_distributions(ctx, kind):
    """Widths from one node block for all samples to one per sample; ties; far outliers."""
    rng = np.random.default_rng(5)
    for n in (120, 500):
        c = clumped(kind, n, rng)
        for sy in (50.0, 0.7, 0.11, 0.02, 1e-3, 1e-7):
            sc, ips, _, st = ctx.periodogram([0, n], c.t, c.y, c.e, FREQS, 0.3, sigma_y=sy,
                                             want_ips=True)
            assert st[0] == 0
            check(c, sc[0], ips[0], 0.3, sy)


def test_scattered_curves_between_others_on_every_entry_point(ctx):
    """Curves that the preparation gives back to the pair sums (every sample alone in its node
    block) next to curves that it keeps, in one call: the results equal each curve's own call,
    from host and device arrays, without allocation, in a search (captured and replayed) and
    through the bands."""
    import torch

    rng = np.random.default_rng(8)
    kinds = ["line", "two", "line", "line", "steps", "line"]
    curves = [clumped(k, n, rng) for k, n in zip(kinds, (400, 330, 260, 300, 150, 20))]
    b = synth.pack(curves)
    kw = dict(sigma_y=2e-4, want_ips=True)
    sc, ips, ipy, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, FREQS, 0.3, **kw)
    assert np.all(st == 0)
    search = dict(f_min=1e-3, f_max=9.0, n_coarse=1500, top_k=4, n_fine=70, sigma_y=2e-4)
    res, coarse = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, want_coarse=True, **search)
    res2, coarse2 = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, want_coarse=True, **search)
    assert res.tobytes() == res2.tobytes() and np.array_equal(coarse, coarse2)
    assert np.all(res["reserved"] == 0)
    bres, trials, scores = ctx.bands_best_period(b.offsets, b.t, b.y, b.e, 0.3, n_trials=20,
                                                 n_grid=4000, sigma_y=2e-4)
    for k, c in enumerate(curves):
        check(c, sc[k], ips[k], 0.3, 2e-4)
        s1, i1, p1, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, FREQS, 0.3, **kw)
        assert np.array_equal(s1[0], sc[k]) and np.array_equal(i1[0], ips[k]) and p1[0] == ipy[k]
        r1, c1 = ctx.best_period([0, c.n], c.t, c.y, c.e, 0.3, want_coarse=True, **search)
        assert r1.tobytes() == res[k:k + 1].tobytes() and np.array_equal(c1[0], coarse[k])
        b1, t1, q1 = ctx.bands_best_period([0, c.n], c.t, c.y, c.e, 0.3, n_trials=20, n_grid=4000,
                                           sigma_y=2e-4)
        assert b1.tobytes() == bres[k:k + 1].tobytes()
        assert np.array_equal(q1[0], scores[k], equal_nan=True)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (b.t, b.y, b.e, FREQS)]
    for call in (ctx.periodogram_dev, ctx.periodogram_noalloc):
        out = torch.zeros((b.n_curves, len(FREQS)), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        pd, sd = call(b.offsets, *dev, out, 0.3, sigma_y=2e-4)
        assert np.array_equal(out.cpu().numpy(), sc) and np.array_equal(pd, ipy)


def test_both_launch_forms_and_mixed_paths_give_the_same_bits(ctx):
    """A batch large enough to run every harmonic group in one wave against single calls that run
    one group per wave, at lengths on both sides of the pair sums, with the sigma_t rule (another
    number of groups for each curve)."""
    curves = [synth.survey_batch_curve(400 + k, n=60 + 23 * k) for k in range(48)]
    b = synth.pack(curves)
    freqs = np.linspace(1e-3, 10.0, 64 * 50 + 5)
    for st in (0.3, qmi.SIGMA_T_SKEWNESS):
        sc, ips, _, _ = ctx.periodogram(b.offsets, b.t, b.y, b.e, freqs, st, want_ips=True)
        for k in (0, 1, 2, 9, 30, 47):
            c = curves[k]
            s1, i1, _, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, freqs, st, want_ips=True)
            assert np.array_equal(s1[0], sc[k]) and np.array_equal(i1[0], ips[k]), (st, k)


def near_tie(r, ref, k, n, sigma_t):
    """The points chosen by two searches of a curve are the same, or differ by no more than the pair
    sums' errors at both, by which near ties are decided: 2 x (1e-7 + 7e-5 / n) of QMI (twice what was
    seen of them, 2e-7 at 617 samples, 4e-7 at 121), the same share of the potentials for nCKP."""
    if r["f_best"] == ref["f_best"][k]:
        return True
    tol = 2 * (1e-7 + 7e-5 / n)
    nckp = tol * (abs(ref["score_nckp"][k]) + 2 / np.sqrt(2 * np.pi) * np.sqrt(n / sigma_t))
    return (abs(r["score"] - ref["score"][k]) <=
            (tol if ref["score"][k] == ref["score_qmi"][k] else nckp) + 2e-7 * abs(r["score"]))


@pytest.mark.parametrize("score", [qmi.SCORE_QMI, qmi.SCORE_NCKP])
@pytest.mark.parametrize("n,count,n_fine", [(96, 200, 1000), (617, 60, 1000), (150, 40, 20000)])
def test_near_ties_are_decided_on_every_path_alike(ctx, score, n, count, n_fine):
    """On flat maxima (neighbouring refined points differ by 1e-6 and less of the score, by 1e-8
    with 20 000 points in a window) a curve's choice is the same alone, in a batch, from device
    arrays and in a replayed graph, and no worse than the FP64 mode's by more than the sums' errors."""
    curves = [synth.survey_batch_curve(500 + k, n=n) for k in range(count)]
    b = synth.pack(curves)
    kw = dict(f_min=1e-3, f_max=2.0, n_coarse=2500, top_k=3, n_fine=n_fine, score=score)
    mixed, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
    ref, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, precision=qmi.PREC_FP64, **kw)
    assert np.all(mixed["reserved"] == 0)
    for k in range(count):
        assert near_tie(mixed[k], ref, k, n, 0.3), (k, mixed[k], ref[k])
    import torch
    dev = ctx.best_period_dev(b.offsets, *[torch.from_numpy(a).cuda() for a in (b.t, b.y, b.e)], 0.3,
                              **kw)
    again, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
    for k in range(0, count, 3):
        c = curves[k]
        one, _ = ctx.best_period([0, c.n], c.t, c.y, c.e, 0.3, **kw)
        for name in ("f_best", "score", "score_nckp", "fine_index", "peak_rank"):
            assert one[0][name] == mixed[k][name] == dev[k][name] == again[k][name], (k, name)


@pytest.mark.parametrize("score", [qmi.SCORE_QMI, qmi.SCORE_NCKP])
@pytest.mark.parametrize("sigma_t,n,n_coarse,n_fine,top_k", [
    (0.3, 97, 4000, 1000, 10),  # about 200 frequencies per window
    (0.3, 617, 4000, 401, 3),  # just enough points to interpolate, and just too few
    (0.3, 617, 4000, 380, 3),
    (0.3, 130, 50000, 41, 10),  # narrow windows, small odd series
    (0.6, 90, 300000, 24, 2),
    (2.0, 64, 2000, 2001, 1),
    (0.1, 400, 4000, 1300, 4),  # 9 groups, about 500 frequencies: both launch forms below
    (0.1, 400, 400, 1000, 2),  # windows too wide: every point is summed
])
def test_interpolated_windows(ctx, sigma_t, n, n_coarse, n_fine, top_k, score):
    """Refined records where the windows' sums are interpolated, against the search in double
    precision, alone and in a batch (the other launch form).  A truncated series is off by at most
    2e-10 of a kernel value per harmonic, far below the sums' own errors: 2e-7 of QMI and of the
    potentials, the bound by which points close to the best are told apart."""
    curves = [synth.survey_batch_curve(500 + k, n=n - (k % 3)) for k in range(40)]
    b = synth.pack(curves)
    kw = dict(f_min=1e-3, f_max=8.0, n_coarse=n_coarse, top_k=top_k, n_fine=n_fine, score=score)
    few = slice(0, int(b.offsets[3]))
    one, _ = ctx.best_period(b.offsets[:4], b.t[few], b.y[few], b.e[few], sigma_t, **kw)
    ref, _ = ctx.best_period(b.offsets[:4], b.t[few], b.y[few], b.e[few], sigma_t,
                             precision=qmi.PREC_FP64, **kw)
    many, _ = ctx.best_period(b.offsets, b.t, b.y, b.e, sigma_t, **kw)
    for r in (one, many):
        for k in range(3):
            assert near_tie(r[k], ref, k, curves[k].n, sigma_t), (k, r[k], ref[k])
            if r["f_best"][k] != ref["f_best"][k]:
                continue
            for s in ("score_qmi", "score_nckp"):
                tol = 2e-7
                if s == "score_nckp":
                    tol *= abs(ref[s][k]) + 2 / np.sqrt(2 * np.pi) * np.sqrt(curves[k].n / sigma_t)
                assert abs(r[s][k] - ref[s][k]) <= tol, (k, s, r[s][k] - ref[s][k])
            assert r["coarse_index"][k] == ref["coarse_index"][k]
    for name in ("f_best", "score", "fine_index"):
        np.testing.assert_array_equal(one[name], many[name][:3])
