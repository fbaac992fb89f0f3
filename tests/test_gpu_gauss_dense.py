"""Direct Gaussian scan of dense series, whose lag lanes lie several samples
apart in the staged window: against the oracle on regular cadences (every lane
at one distance) and random times, with the window range filling the stage and
past it (mixed c 1e-5, b 1e-6; FP64 c 1e-11, b 1e-12, as in
test_gpu_gauss_scan.py; b against sums in extended precision: on a regular
cadence the oracle adds equal terms 6000 times and is itself 1.1e-12 off); and the time of a call whose lanes are eight samples
apart beside that of the same weights with lanes one sample apart.
"""
import functools
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu

N, K = 6000, 70
TOL = {"mixed": (1e-5, 1e-6), "fp64": (1e-11, 1e-12)}


@functools.lru_cache(maxsize=None)
def _pairs(dens, step, regular):
    """The pair count b of every lag, summed in extended precision."""
    t, lags, h = _times(dens, step, regular)[0], step * np.arange(K), 0.5
    b = []
    for lag in lags:
        c = t + lag
        lo = np.searchsorted(t, c - 6.0 * h, "left")
        hi = np.searchsorted(t, c + 6.0 * h, "left")
        i = lo[:, None] + np.arange(max(1, int((hi - lo).max())))
        d = (t[np.minimum(i, t.size - 1)] - c[:, None]) / h
        w = np.where(i < hi[:, None], np.exp(-0.5 * d * d), 0.0)
        b.append(float(w.sum(dtype=np.longdouble) / (np.sqrt(2.0 * np.pi) * h)))
    return np.array(b)


def _times(dens, step, regular):
    rng = synth.rng_for(int(dens * 10 + step))
    return (np.arange(N) / dens if regular else np.sort(rng.uniform(0.0, N / dens, N))), rng


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("errors", [False, True])
# samples per unit of time, lag step: ranges of about 64 step dens + 12 h dens
@pytest.mark.parametrize("dens,step,regular", [(8.0, 1.0, True), (16.0, 0.5, False),
                                               (16.0, 0.86, True), (16.0, 1.36, False),
                                               (32.0, 1.0, True)])
def test_direct_dense(dens, step, regular, errors, precision):
    print(f"case: gauss dense={dens} step={step} errors={errors} {precision}", flush=True)
    h = 0.5
    t, rng = _times(dens, step, regular)
    x = np.sin(t / 9.0) + 0.3 * rng.normal(size=N)
    err = rng.uniform(0.5, 1.5, N) if errors else None
    lags = step * np.arange(K)
    st, oc, _, _ = O.acf(t, x, lags, "gaussian", h, err=err)
    assert st == 0
    c, b, _, _ = ncf.acf(t, x, lags, "gaussian", h, err=err, precision=precision, method="direct")
    ct, bt = TOL[precision]
    np.testing.assert_allclose(c, oc, rtol=0, atol=ct)
    np.testing.assert_allclose(b, _pairs(dens, step, regular), rtol=bt, atol=0)


def _best(f, torch, n=12):
    f()
    ts = []
    for _ in range(n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return min(ts)


@pytest.mark.parametrize("errors", [False, True])
def test_lanes_far_apart_take_no_longer(errors):
    """The same windows at lags one sample and eight samples apart: the wider
    range costs a little staging (1.1 to 1.2 times so; 1.6 to 1.7 with the samples as
    records, whose reads conflict)."""
    import torch
    print(f"case: gauss dense, time, errors={errors}", flush=True)
    rng = synth.rng_for(3)
    n, dens = 100_000, 16.0
    dev = torch.device("cuda:0")
    t = np.sort(rng.uniform(0.0, n / dens, n))
    x = torch.as_tensor(np.sin(t / 9.0) + 0.3 * rng.normal(size=n), device=dev)
    err = torch.as_tensor(rng.uniform(0.5, 1.5, n), device=dev) if errors else None
    t = torch.as_tensor(t, device=dev)

    def of(step):
        lags = step * torch.arange(256.0, dtype=torch.float64, device=dev)
        return _best(lambda: ncf.acf(t, x, lags, "gaussian", 0.5, err=err, method="direct"), torch)

    near, far = of(1.0 / 16.0), of(0.5)
    print(f"near {near * 1e6:.0f} us, far {far * 1e6:.0f} us, ratio {far / near:.2f}", flush=True)
    assert far <= 1.5 * near
