"""The ACF spread inside the first transform pass against the separate kernels: the
same series in a batch of 512 spreading tiles of its transform size, which takes
the fused pass, and alone, which does not (the kernels that ran are checked). Every
first radix from 2 to 256 (sizes 2^13 to 2^20), seasonal gaps, a lone far sample
and a series of several samples per cell, lags on a lattice (folded spectrum) and
off it (inverse transform). Mixed: the same operations in the same order, bit for
bit. FP64: the passes truncate the kernel at other cells (each below its target of
1e-13) and the lags kept have 0.01 of the reference pair count or more: 1e-10.
"""
import numpy as np
import pytest

from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


def _series(rng, span, i):
    """About 0.6 samples a day over `span` days, i picks the sampling."""
    if i == 1:  # clustered in a fifth of the span, and one sample far away
        t = np.sort(rng.uniform(0.0, 0.2 * span, int(0.3 * span)))
        t[-1] = span
    elif i == 2:  # several samples per grid cell
        t = np.sort(rng.uniform(0.0, span, int(20 * span)))
    else:  # seasons of 250 days, or evenly spread
        t = np.sort(rng.uniform(0.0, span, int(0.9 * span)))
        if i % 2 == 0:
            t = t[(t % 365.0) < 250.0]
    t[0], t[-1] = 0.0, span
    return t


def _span(lg, lags, lattice, precision):
    """A span in days that the planner gives a grid of 2^lg cells."""
    for days in np.arange(2.4, 0.3, -0.05) * 19_000.0 * 2.0 ** (lg - 17):
        _, _, n, _, p = ncf.diag_grid(0.0, days, lags, 0.5, precision=precision)
        if n == 2 ** lg and (p > 0) == lattice:
            return float(days)
    raise AssertionError(f"no span for 2^{lg} cells")


def _kernels(f):
    ncf.profile_enable(True)
    try:
        r = f()
        return r, set(ncf.profile_read())
    finally:
        ncf.profile_enable(False)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("lattice", [True, False])
@pytest.mark.parametrize("lg", range(13, 21))
def test_batch_and_single(lg, lattice, precision):
    print(f"case: spread routes 2^{lg} lattice={lattice} {precision}", flush=True)
    rng = synth.rng_for(lg)
    count = max(2, 2 ** (21 - lg))
    lags = np.arange(40.0) if lattice else np.arange(40.0) ** 1.02
    span = _span(lg, lags, lattice, precision)
    kw = dict(kernel="gaussian", h=0.5, precision=precision, spectral_always=True)
    ts = [_series(rng, span, min(i, 3 + i % 2)) for i in range(count)]
    xs = [np.sin(t / 9.0) + 0.5 * rng.normal(size=t.size) for t in ts]
    offs = np.concatenate([[0], np.cumsum([t.size for t in ts])])
    fused = "spread_fft_f32" if precision == "mixed" else "spread_fft_f64"
    apart = "spread_f32" if precision == "mixed" else "spread_f64"
    (c, b, _, st, _), ran = _kernels(lambda: ncf.acf_batch(offs, np.concatenate(ts),
                                                           np.concatenate(xs), lags, **kw))
    assert (st == 0).all()
    assert fused in ran and apart not in ran, ran
    for i in range(min(count, 5)):
        (c1, b1, _, _), ran = _kernels(lambda: ncf.acf(ts[i], xs[i], lags, **kw))
        assert apart in ran and fused not in ran, ran
        if precision == "mixed":
            np.testing.assert_array_equal(c[i], c1)
            np.testing.assert_array_equal(b[i], b1)
        else:
            np.testing.assert_allclose(c[i], c1, rtol=0, atol=1e-10)
            np.testing.assert_allclose(b[i], b1, rtol=1e-10, atol=0)
