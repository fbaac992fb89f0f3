"""Lattice batch of one sample per cell, the ordinary case: the sample-index table
costs less than the moments pass, which reads twice its bytes, and the first passes
no more than 1.4 times the last pass, product and inverse (the samples of a cell
past the first are read only where it has them); and its sums against the oracle.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


def test_one_sample_per_cell():
    import torch
    print("case: lattice batch, one sample per cell", flush=True)
    dev = torch.device("cuda:0")
    nser, n, lags = 600, 65000, np.arange(200.0)
    rng = synth.rng_for(65)
    t = np.tile(np.arange(float(n)), nser)
    x = np.sin(t / 9.0) + 0.5 * rng.normal(size=t.size)
    d = [torch.as_tensor(a, device=dev) for a in (t, x, lags)]
    offs = n * np.arange(nser + 1)

    def call():
        return ncf.acf_regular_batch(offs, d[0], d[1], d[2], 1.0, "rectangle", 0.5)

    out = call()
    took = {}
    ncf.profile_enable(True)
    try:
        total = {}
        for _ in range(5):
            call()
            now = {k: r["total_ms"] for k, r in ncf.profile_read().items()}
            for k, v in now.items():
                took[k] = min(took.get(k, 1e9), v - total.get(k, 0.0))
            total = now
    finally:
        ncf.profile_enable(False)
    first = sum(v for k, v in took.items() if k.startswith("reg_first"))
    print(f"ratio table {took['reg_seg'] / took['moments']:.2f}, "
          f"first pass {first / took['reg_mid']:.2f}", flush=True)
    st, oc, ob, _ = O.acf(t[:4000], x[:4000], lags[:50], "rectangle", 0.5)
    assert st == 0
    c, b = ncf.acf_regular(d[0][:4000], d[1][:4000], d[2][:50], 1.0, "rectangle", 0.5)[:2]
    np.testing.assert_allclose(c.cpu().numpy(), oc, rtol=0, atol=1e-10)
    np.testing.assert_array_equal(b.cpu().numpy(), ob)
    np.testing.assert_array_equal(out[1][0].cpu().numpy(), n - lags)
    assert took["reg_seg"] <= 0.95 * took["moments"]
    assert first <= 1.4 * took["reg_mid"]


# lag workgroups (6 per series) on either side of one per CU and of two per CU
@pytest.mark.parametrize("few,many,n", [(42, 43, 3000), (84, 88, 20000)])
def test_lag_workgroups(few, many, n):
    import torch
    print(f"case: lags of {few} and {many} lattice series", flush=True)
    dev = torch.device("cuda:0")
    lags = torch.arange(366.0, dtype=torch.float64, device=dev)
    took = []
    for nser in (few, many):
        rng = synth.rng_for(nser)
        t = np.tile(np.arange(float(n)), nser)
        x = np.sin(t / 9.0) + 0.5 * rng.normal(size=t.size)
        t, x = (torch.as_tensor(a, device=dev) for a in (t, x))
        offs = n * np.arange(nser + 1)
        best, before = 1e9, 0.0
        ncf.profile_enable(True)
        ncf.profile_filter("reg_lags")
        try:
            for _ in range(8):
                out = ncf.acf_regular_batch(offs, t, x, lags, 1.0, "rectangle", 0.5)
                total = ncf.profile_read()["reg_lags"]["total_ms"]
                best, before = min(best, total - before), total
        finally:
            ncf.profile_enable(False)
            ncf.profile_filter(None)
        took.append(best)
        for i in (0, nser - 1):
            c, b = ncf.acf_regular(t[:n], x[i * n:(i + 1) * n], lags, 1.0, "rectangle", 0.5)[:2]
            assert float((out[0][i] - c).abs().max()) <= 1e-12
            assert bool((out[1][i] == b).all())
    print(f"ratio {took[0] / took[1]:.2f}", flush=True)
    assert took[0] <= 1.15 * took[1]
