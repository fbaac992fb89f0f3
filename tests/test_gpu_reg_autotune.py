"""Autotuned plans of lattice series: the transform variants are timed only where a
series takes the general route, the one that reads them, and the plan agrees with
the plain call (c 1e-11).
"""
import numpy as np
import pytest

from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


# dense lattices are fused; weights, and a series of few samples, are not
@pytest.mark.parametrize("errors,sparse,candidates", [(False, False, 1), (True, False, 3),
                                                      (False, True, 3)])
def test_candidates(errors, sparse, candidates):
    print(f"case: lattice autotune errors={errors} sparse={sparse}", flush=True)
    rng = synth.rng_for(12)
    ts = [synth.lattice_times(rng, n, keep=0.9) for n in (3000, 9000)]
    if sparse:
        ts.append(np.cumsum(rng.integers(20, 60, 200)).astype(float))
    offs = np.concatenate([[0], np.cumsum([t.size for t in ts])])
    t = np.concatenate(ts)
    x = rng.normal(size=t.size)
    err = rng.uniform(0.5, 1.5, t.size) if errors else None
    lags = np.arange(50.0)
    plan = ncf.plan_acf_regular(offs, t, lags, 1.0, "gaussian", 2.0, err=err, autotune=True)
    try:
        info = plan.info()
        assert info["autotuned"] == 1 and info["candidates"] == candidates, info
        c = plan.execute(x)[0]
    finally:
        plan.close()
    r = ncf.acf_regular_batch(offs, t, x, lags, 1.0, "gaussian", 2.0, err=err)[0]
    np.testing.assert_allclose(c, r, rtol=0, atol=1e-11)
