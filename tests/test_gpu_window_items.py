"""Items of a window launch of middle size: a few rounds of the chip, not one of
its rounds part-filled (3072 for the Gaussian, 1434 of up to 2048 workgroups for the
rectangle, whose items are shorter for it than the range allows), and the sums of
such items against the oracle, on even times and on bursts.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bursts", [0, 9])
@pytest.mark.parametrize("kernel,n,lags,least,most", [("gaussian", 20000, 256, 2600, 4096),
                                                      ("rectangle", 31000, 324, 1300, 2048)])
def test_middle_launch(kernel, n, lags, least, most, bursts):
    import torch
    print(f"case: window items, {kernel}, {bursts} bursts", flush=True)
    dev = torch.device("cuda:0")
    rng = synth.rng_for(n + bursts)
    t = rng.uniform(0.0, n, n)
    if bursts:
        t = n / bursts * rng.integers(0, bursts, n) + rng.uniform(0.0, n / bursts / 4, n)
    t = np.sort(t)
    x = np.sin(t / 9.0) + 0.5 * rng.normal(size=n)
    lg = np.arange(float(lags))
    dt, dx, dl = (torch.as_tensor(a, device=dev) for a in (t, x, lg))
    p = ncf.plan_acf(np.array([0, n]), dt, dl, kernel, 0.5, method="direct")
    items = p.info()["window_items"]
    p.close()
    c, b = ncf.acf(dt, dx, dl, kernel, 0.5, method="direct")[:2]
    st, oc, ob, _ = O.acf(t, x, lg, kernel, 0.5)
    assert st == 0
    live = ob > 0  # (bursts leave lags without a pair)
    np.testing.assert_allclose(c.cpu().numpy()[live], oc[live], rtol=0, atol=1e-5)
    np.testing.assert_allclose(b.cpu().numpy(), ob, rtol=1e-6, atol=0)
    print(f"ratio items {items}", flush=True)
    assert bursts or least <= items <= most
