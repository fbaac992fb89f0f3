"""FP64 Gaussian scan with windows of 0 to 13 samples, which it takes by twos
from the staged range and by fours from global memory: clusters of samples that
each fill one window, at lags that meet every pair of sizes, in calls whose
window range fits the stage and in calls whose range does not, against the
oracle (c 1e-11, b 1e-12, as in test_gpu_gauss_scan.py).
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("errors", [False, True])
# lags 10 apart over 30 (staged), and 64 of them over thousands of samples (not)
@pytest.mark.parametrize("K", [3, 64, 300])
@pytest.mark.parametrize("clusters", [40, 900])
def test_small_windows(clusters, K, errors):
    print(f"case: gauss fp64 clusters={clusters} K={K} errors={errors}", flush=True)
    rng = synth.rng_for(clusters + K)
    size = rng.integers(0, 14, clusters)
    size[:14] = np.arange(14)
    at = np.repeat(10.0 * np.arange(clusters), size)
    t = np.sort(at + rng.uniform(-0.2, 0.2, at.size))
    x = rng.normal(size=t.size)
    err = rng.uniform(0.5, 1.5, t.size) if errors else None
    lags = 10.0 * np.arange(K)
    for h in (0.2, 0.05):  # whole clusters; parts of them
        st, oc, ob, _ = O.acf(t, x, lags, "gaussian", h, err=err)
        assert st == 0
        c, b, _, _ = ncf.acf(t, x, lags, "gaussian", h, err=err, precision="fp64",
                             method="direct")
        np.testing.assert_allclose(c, oc, rtol=0, atol=1e-11)
        np.testing.assert_allclose(b, ob, rtol=1e-12, atol=0)
