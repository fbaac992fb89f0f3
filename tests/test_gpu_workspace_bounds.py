"""Calls whose first plan does not fit the workspace bound: the window scan takes
fewer, longer items, in two steps (a bound that items sized series by series
fitted is enough for the first: 76 MB here), and the ACF spread gives up the
sample-index tables of its fused form. What was planned is read off the call's log
line and its kernels; results against the oracle (c 1e-5, b 1e-6) and, for the
spread, bit for bit against the call without a bound. The bound is read once per
process: each case runs in one of its own.
"""
import json
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASE = textwrap.dedent("""
    import hashlib, json, sys
    sys.path.insert(0, ".")
    import numpy as np
    import torch
    from oracle import oracle as O
    from paper_2609_03866_amd import ncf, synth
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")
    rng = synth.rng_for(8)
    kernel = "rectangle" if sys.argv[1] == "rectangle" else "gaussian"
    if sys.argv[1] != "spread":  # 2000 series of 1600, ranges of about 640 samples
        ns, n, kw = 2000, 1600, dict(method="direct")
        t = np.sort(rng.uniform(0.0, n, (ns, n)), axis=1)
        lags = 10.0 * np.arange(64)
    else:  # 128 grids of 2^17 cells: their tables take 4 MB
        ns, n, kw = 128, 20_000, dict(spectral_always=True)
        t = np.arange(n) + rng.uniform(0.0, 0.3, (ns, 1))
        lags = np.arange(100.0)
    x = np.sin(t / 9.0) + 0.5 * rng.normal(size=t.shape)
    ncf.profile_enable(True)
    c, b, k, st, rc = ncf.acf_batch(n * np.arange(ns + 1), dev(t.ravel()), dev(x.ravel()),
                                    dev(lags), kernel, 0.5, raise_on_error=False, **kw)
    if rc == 0:
        c, b = c.cpu().numpy(), b.cpu().numpy()
        for i in (0, ns - 1) if sys.argv[1] != "spread" else ():
            _, oc, ob, ok = O.acf(t[i], x[i], lags, kernel, 0.5)
            assert kernel == "gaussian" or np.array_equal(k[i].cpu().numpy(), ok)
            assert np.max(np.abs(c[i] - oc)) <= 1e-5
            assert np.max(np.abs(b[i] / ob - 1.0)) <= 1e-6
    print("RESULT " + json.dumps(dict(rc=int(rc), kernels=sorted(ncf.profile_read()),
                                      sha=hashlib.sha256(c.tobytes() + b.tobytes()).hexdigest()
                                      if rc == 0 else "")))
""")


def _run(what, mb):
    env = dict(os.environ, NCF_LOG="1")
    env.pop("NCF_WORKSPACE_LIMIT_MB", None)
    if mb:
        env["NCF_WORKSPACE_LIMIT_MB"] = str(mb)
    r = subprocess.run([sys.executable, "-c", CASE, what], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=240)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    out = json.loads(r.stdout.split("RESULT ", 1)[1])
    out["items"] = [int(w.split("=")[1]) for w in r.stderr.split() if w.startswith("window_items=")]
    return out


# tiles of 112 samples and of 64: 15 and 25 per series, 16384 items by grouping
@pytest.mark.parametrize("mb,items", [(0, 30_000), (76, 16_000), (62, 2000)])
def test_window_items(mb, items):
    print(f"case: window items under {mb} MB", flush=True)
    r = _run("gaussian", mb)
    assert r["rc"] == 0 and r["items"][-1] == items, r


def test_rectangle_items():
    print("case: rectangle items under 95 and 85 MB", flush=True)
    rs = [_run("rectangle", mb) for mb in (0, 95, 85)]
    assert [r["rc"] for r in rs] == [0, 0, 0]
    assert rs[0]["items"][-1] > rs[1]["items"][-1] > rs[2]["items"][-1] == 2000, rs


def test_fused_spread_without_tables():
    print("case: fused spread, bound below its index tables", flush=True)
    free, bound = _run("spread", 0), _run("spread", 228)
    assert "spread_fft_f32" in free["kernels"]
    assert "spread_f32" in bound["kernels"] and "spread_fft_f32" not in bound["kernels"]
    assert free["rc"] == 0 and bound["rc"] == 0
    assert free["sha"] == bound["sha"]
