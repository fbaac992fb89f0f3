"""Outer tiles of a window scan: a batch whose series are a little longer than
one tile takes no longer than in proportion to one whose series fill it (a short
last tile at the same place in every series leaves half the CUs with the long
ones: 1.7 to 1.8 times); and its sums against the oracle.
"""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


def _best(f, torch, n=8):
    f()
    ts = []
    for _ in range(n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return min(ts)


# the longest single tile, and a series just past it
@pytest.mark.parametrize("errors,full,past", [(True, 432, 448), (False, 688, 704)])
def test_short_last_tile(errors, full, past):
    import torch
    print(f"case: window tiles {full} and {past}, errors={errors}", flush=True)
    dev = torch.device("cuda:0")
    nser, lags = 4000, np.arange(128.0)
    took = []
    for n in (full, past):
        rng = synth.rng_for(n)
        t = np.sort(rng.uniform(0.0, n, (nser, n)), axis=1)
        x = np.sin(t / 9.0) + 0.5 * rng.normal(size=t.shape)
        e = rng.uniform(0.5, 1.5, t.shape) if errors else None
        d = [torch.as_tensor(a.ravel(), device=dev) if a is not None else None for a in (t, x, e)]
        lg = torch.as_tensor(lags, device=dev)
        offs = n * np.arange(nser + 1)
        out = []

        def call():
            out[:] = ncf.acf_batch(offs, d[0], d[1], lg, "gaussian", 0.5, err=d[2],
                                   method="direct")

        took.append(_best(call, torch))
        for i in (0, nser - 1):
            st, oc, ob, _ = O.acf(t[i], x[i], lags, "gaussian", 0.5,
                                  err=e[i] if errors else None)
            assert st == 0
            np.testing.assert_allclose(out[0][i].cpu().numpy(), oc, rtol=0, atol=1e-5)
            np.testing.assert_allclose(out[1][i].cpu().numpy(), ob, rtol=1e-6, atol=0)
    print(f"ratio {took[1] / took[0]:.2f}", flush=True)
    assert took[1] <= 1.35 * took[0]
