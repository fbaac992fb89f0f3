"""Window scans of few lags: an item has a run of outer samples for each lane that
the lags leave, whatever the length of its tile (tiles shorter than the number of
runs, longer ones, a part-filled last round), and two lags of a dense series take
no longer than 32 of them. The sums are checked against the oracle.
"""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lags", [1, 2, 3, 10, 33])
@pytest.mark.parametrize("kernel,precision", [("gaussian", "mixed"), ("gaussian", "fp64"),
                                              ("rectangle", "mixed")])
def test_few_lags(kernel, precision, lags):
    import torch
    print(f"case: {lags} lags, {kernel} {precision}", flush=True)
    dev = torch.device("cuda:0")
    lg = np.arange(lags) - 0.5 * (lags > 2)
    for n, bursts, errors in ((40, 0, False), (257, 0, True), (2338, 6, False), (2338, 0, True)):
        rng = synth.rng_for(1000 * lags + n + bursts)
        t = rng.uniform(0.0, n / 3.0, n)
        if bursts:
            t = n / 3.0 / bursts * rng.integers(0, bursts, n) + rng.uniform(0.0, 12.0, n)
        t = np.sort(t)
        x = np.sin(t / 5.0) + 0.4 * rng.normal(size=n)
        e = rng.uniform(0.5, 1.5, n) if errors else None
        d = [torch.as_tensor(a, device=dev) if a is not None else None for a in (t, x, lg, e)]
        c, b = ncf.acf(d[0], d[1], d[2], kernel, 0.5, err=d[3], method="direct",
                       precision=precision)[:2]
        st, oc, ob, _ = O.acf(t, x, lg, kernel, 0.5, err=e)
        assert st == 0
        fp64 = precision == "fp64"
        np.testing.assert_allclose(c.cpu().numpy(), oc, rtol=0, atol=1e-10 if fp64 else 1e-5)
        np.testing.assert_allclose(b.cpu().numpy(), ob, rtol=1e-11 if fp64 else 1e-6, atol=0)


@pytest.mark.parametrize("n", [2400, 6000])
def test_two_lags_time(n):
    import torch
    print(f"case: two lags and 32, {n} samples", flush=True)
    dev = torch.device("cuda:0")
    rng = synth.rng_for(n)
    t = np.sort(rng.uniform(0.0, n / 20.0, n))
    t, x = (torch.as_tensor(a, device=dev) for a in (t, np.sin(t)))

    def best(lags):
        lg = torch.arange(lags, dtype=torch.float64, device=dev)
        took = []
        for _ in range(12):
            torch.cuda.synchronize()
            s = time.perf_counter()
            ncf.acf(t, x, lg, "gaussian", 2.0, method="direct", precision="fp64")
            torch.cuda.synchronize()
            took.append(time.perf_counter() - s)
        return min(took)

    few, many = best(2), best(32)
    print(f"ratio {few / many:.2f}", flush=True)
    assert few <= many
