"""Gaps in a regular lattice: the sample-index table of the fused route fills
the entries of a gap (8 cells each) by the lane up to 32, by the wave up to
4096, by the workgroup beyond. Gaps on either side of both limits, before the
first sample of a chunk of 2048 and inside one, several in one chunk, and the
largest that the route's sample limit allows, against the oracle (c 1e-9, counts
exact, as in test_gpu_regular.py); and the time of a call on two campaigns
beside that of as many samples spread over the same lattice.
"""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


def _check(t, lags):
    x = synth.rng_for(t.size).normal(size=t.size)
    c, b, k, _ = ncf.acf_regular(t, x, lags, 1.0, "rectangle", 1.5)
    st, oc, ob, ok = O.acf_regular(t, x, lags, 1.0, "rectangle", 1.5)
    assert st == 0
    np.testing.assert_allclose(c, oc, rtol=0, atol=1e-9)
    np.testing.assert_array_equal(k, ok)


@pytest.mark.parametrize("cells", [255, 256, 263, 264, 272, 8 * 4095, 8 * 4096 + 1, 8 * 4097,
                                   70_001])
@pytest.mark.parametrize("at", [1, 700, 2047, 2048, 2049])
def test_one_gap(cells, at):
    print(f"case: lattice gap of {cells} cells after {at} samples", flush=True)
    n = max(4500, cells // 16 + 4500)
    t = np.arange(n) + np.where(np.arange(n) >= at, cells, 0)
    _check(t.astype(float), np.concatenate([np.arange(40.0), [1500.0]]))


def test_many_gaps():
    """Wide gaps in turn with runs: fourteen of the workgroup's in one chunk."""
    print("case: lattice, fourteen gaps past 4096 entries", flush=True)
    step = np.ones(70_000)
    step[30:1900:134] = 8 * 4096 + 8 * np.arange(14) + 3
    step[2100:4000:37] = 300
    _check(np.cumsum(step), np.arange(50.0))


def _best(f, torch, n=20):
    f()
    ts = []
    for _ in range(n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
    return min(ts)


def test_two_campaigns_take_no_longer():
    """66,000 samples of one minute in two campaigns 975,000 minutes apart, and
    spread over the same span: the same transforms (1.1 times the time; one lane
    filling the gap: 31 times)."""
    import torch
    print("case: lattice, two campaigns, time", flush=True)
    rng = synth.rng_for(9)
    n, G = 66_000, 1_040_000
    dev = torch.device("cuda:0")
    lags = torch.arange(100.0, dtype=torch.float64, device=dev)
    x = torch.as_tensor(rng.normal(size=n), device=dev)

    def of(m):
        t = torch.as_tensor(m.astype(np.float64), device=dev)
        return _best(lambda: ncf.acf_regular(t, x, lags, 1.0, "rectangle", 0.5), torch)

    two = np.concatenate([np.arange(n // 2), G - n // 2 + np.arange(n // 2)])
    spread = np.sort(rng.choice(G - 2, n - 2, replace=False) + 1)
    spread = np.concatenate([[0], spread, [G - 1]])
    assert of(two) <= 4.0 * of(spread)
