"""Curves that the preparation gives back to the pair sums share one more section, wherever they stand
in a batch: every other curve, all, the first, the last; results small and large (fetched at once, or
after that section); every entry point.  The results are each curve's own, bit for bit, and the
launches that form sums do not grow with the number of given-back curves."""
import numpy as np
import pytest
import torch

from paper_1412_1840_amd import qmi, synth

pytestmark = pytest.mark.gpu

SY = 1.0


def curve(k, n, scattered):
    rng = np.random.default_rng(k)
    c = synth.survey_batch_curve(k, n=n)
    return synth.Curve(c.t, rng.uniform(0, 5000.0 if scattered else 12.0, n), c.e, False)


def batch(pattern, n, count):
    take = {"every other": lambda k: k % 2 == 1, "all": lambda k: True, "first": lambda k: k == 0,
            "last": lambda k: k == count - 1}[pattern]
    return [curve(k, n - k % 3, take(k)) for k in range(count)]


def launches(ctx):
    return ctx.stats()["pair_launches"]


@pytest.mark.parametrize("precision,n", [(qmi.PREC_MIXED, 130), (qmi.PREC_FP64, 260)])
@pytest.mark.parametrize("pattern", ["every other", "all", "first", "last"])
def test_periodograms(pattern, precision, n):
    curves = batch(pattern, n, 40)
    b = synth.pack(curves)
    with qmi.Context(0) as ctx:
        ctx.set_option(qmi.OPT_USE_GRAPH, 0)
        for n_freq in (9, 7001):  # 7001 x 40 x 8 bytes: over 2 MB
            f = np.linspace(1e-3, 9.0, n_freq)
            kw = dict(sigma_y=SY, precision=precision)
            sc, ips, ipy, st = ctx.periodogram(b.offsets, b.t, b.y, b.e, f, 0.3, want_ips=True, **kw)
            assert launches(ctx) == 2 and np.all(st == 0)
            dev = [torch.from_numpy(a).cuda() for a in (b.t, b.y, b.e, f)]
            out = torch.zeros((len(curves), n_freq), dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            for call in (ctx.periodogram_dev, ctx.periodogram_noalloc):
                out.zero_()
                torch.cuda.synchronize()
                y1, st = call(b.offsets, *dev, out, 0.3, **kw)
                assert np.array_equal(out.cpu().numpy(), sc) and np.array_equal(y1, ipy)
            for k in (0, 1, 2, 17, 38, 39):
                c = curves[k]
                s1, i1, y1, _ = ctx.periodogram([0, c.n], c.t, c.y, c.e, f, 0.3, want_ips=True, **kw)
                assert np.array_equal(s1[0], sc[k]) and np.array_equal(i1[0], ips[k])
                assert y1[0] == ipy[k]


@pytest.mark.parametrize("n_coarse", [600, 9001])
@pytest.mark.parametrize("pattern", ["every other", "all", "last"])
def test_searches(pattern, n_coarse):
    curves = batch(pattern, 130, 40)
    b = synth.pack(curves)
    kw = dict(f_min=1e-3, f_max=9.0, n_coarse=n_coarse, top_k=3, n_fine=1000, sigma_y=SY)
    with qmi.Context(0) as ctx:
        res, coarse = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, want_coarse=True, **kw)
        again, coarse2 = ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, want_coarse=True, **kw)
        assert res.tobytes() == again.tobytes() and np.array_equal(coarse, coarse2)
        assert np.all(res["reserved"] == 0) and np.all(res["status"] == 0)
        out = torch.zeros((len(curves), n_coarse), dtype=torch.float64, device="cuda")
        dev = ctx.best_period_dev(b.offsets, *[torch.from_numpy(a).cuda() for a in (b.t, b.y, b.e)],
                                  0.3, coarse_out=out, **kw)
        assert dev.tobytes() == res.tobytes() and np.array_equal(out.cpu().numpy(), coarse)
        ctx.set_option(qmi.OPT_USE_GRAPH, 0)
        ctx.best_period(b.offsets, b.t, b.y, b.e, 0.3, **kw)
        assert launches(ctx) == 4  # the grid and the windows, twice
        bres, trials, scores = ctx.bands_best_period(b.offsets, b.t, b.y, b.e, 0.3, n_trials=50,
                                                     n_grid=4000, sigma_y=SY)
        assert launches(ctx) == 2
        for k in (0, 1, 2, 17, 38, 39):
            c = curves[k]
            r1, c1 = ctx.best_period([0, c.n], c.t, c.y, c.e, 0.3, want_coarse=True, **kw)
            assert r1.tobytes() == res[k:k + 1].tobytes() and np.array_equal(c1[0], coarse[k]), k
            b1, t1, q1 = ctx.bands_best_period([0, c.n], c.t, c.y, c.e, 0.3, n_trials=50,
                                               n_grid=4000, sigma_y=SY)
            assert b1.tobytes() == bres[k:k + 1].tobytes()
            assert np.array_equal(t1[0], trials[k], equal_nan=True)
            assert np.array_equal(q1[0], scores[k], equal_nan=True)
