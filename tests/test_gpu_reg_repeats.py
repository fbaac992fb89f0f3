"""Repeated times on a regular lattice: runs of 1 to 13 samples in a cell (the
lane of the first reads four at a time) and longer ones, the sample count on
either side of the fused route's limit of four per cell, series of one tile
beyond it, and the weighted mode, against the oracle (c 1e-9, counts exact);
and the route that each takes.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_03866_amd import ncf, synth

pytestmark = pytest.mark.gpu


def _series(G, per, rng):
    t = np.sort(np.concatenate([np.arange(G), rng.integers(0, G, G * per - G)]))
    return t.astype(float)


@pytest.mark.parametrize("errors", [False, True])
@pytest.mark.parametrize("G,runs", [(600, range(1, 14)), (6000, range(1, 9)), (6000, [1, 2, 3]),
                                    (300, [1, 130])])
def test_runs(G, runs, errors):
    print(f"case: lattice runs G={G} {list(runs)} errors={errors}", flush=True)
    rng = synth.rng_for(G)
    t = np.repeat(np.arange(G), np.resize(list(runs), G)).astype(float)
    x = rng.normal(size=t.size)
    err = rng.uniform(0.5, 2.0, t.size) if errors else None
    lags = np.arange(40.0)
    c, b, k, _ = ncf.acf_regular(t, x, lags, 1.0, "rectangle", 1.5, err=err)
    st, oc, ob, ok = O.acf_regular(t, x, lags, 1.0, "rectangle", 1.5, err=err)
    assert st == 0
    np.testing.assert_allclose(c, oc, rtol=0, atol=1e-9)
    np.testing.assert_array_equal(k, ok)


@pytest.mark.parametrize("G,per,fused", [(6000, 1, True), (6000, 4, True), (6000, 5, False),
                                         (60_000, 8, False), (2000, 16, True)])
def test_route(G, per, fused):
    """Above four samples per cell the general route's fill has four times the
    workgroups (60,000 cells, 8 per cell: fused 310 us, general 187); a transform
    of one tile is faster fused at any count."""
    print(f"case: lattice route G={G} per={per}", flush=True)
    rng = synth.rng_for(G + per)
    t = _series(G, per, rng)
    x = rng.normal(size=t.size)
    ncf.profile_enable(True)
    try:
        ncf.acf_regular(t, x, np.arange(20.0), 1.0, "rectangle", 0.5)
        names = set(ncf.profile_read())
    finally:
        ncf.profile_enable(False)
    assert ("reg_first" in names) == fused, names
    assert ("reg_fill" in names) == (not fused), names
