"""The kernels that add the regions' split sums, at region counts and sizes where their waits for memory decide: many small
closed regions (one split each), regions of several splits, empty ones between; values against each region alone, and the
time of the four sums of dL/dQ against that of F's one (with one sum after the other it was three times as long)."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, host, maxrel, step

pytestmark = pytest.mark.gpu


def _boxes(n, sub):
    """n boxes side by side, each subdivided `sub` times (12 * 4^sub faces), and their face offsets."""
    v, t = mg.box(6.0, 7.0, 8.0)
    for _ in range(sub):
        v, t = mg.subdivide(v, t)
    rng = np.random.default_rng(n + sub)
    vs = [v + rng.uniform(-50.0, 50.0, 3) for _ in range(n)]
    return np.concatenate(vs), np.concatenate([t + len(v) * i for i in range(n)]), [len(t) * i for i in range(n + 1)]


def _grads(v, t, off, rho, q, c, mode, **kw):
    return pft.backward_3d_regions(dev(v), dev(t, torch.int32), off, dev(np.asarray(rho)), q, c, mode=mode, **kw)


@pytest.mark.parametrize("mode,tol", [("fp64", 1e-11), ("fp32c", 2e-5)])
def test_values(gpu, mode, tol):
    """Three regions of 1, 3 and 12 splits and empty ones about them: the sums are those of each region alone."""
    parts = [_boxes(1, s) for s in (1, 2, 3)]
    nv = np.cumsum([0] + [len(p[0]) for p in parts])
    v, t = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + nv[i] for i, p in enumerate(parts)])
    ends = np.cumsum([len(p[1]) for p in parts])
    off = [0, 0, int(ends[0]), int(ends[0]), int(ends[0]), int(ends[1]), int(ends[2]), int(ends[2])]
    rho = [3.0, 1.0, 5.0, -2.0, 0.7, 1.3, 9.0]
    rng = np.random.default_rng(1)
    q = dev(mg.q_random_ball(300, 0.5, rng))
    c = dev(rng.normal(size=300) + 1j * rng.normal(size=300))
    step(f"regions with empty ones {mode}")
    gv, gr, gq = (host(x) for x in _grads(v, t, off, rho, q, c, mode))
    want_q, want_r, want_v = 0.0, np.zeros(7), np.zeros_like(v)
    for i, j in enumerate((1, 4, 5)):
        step(f"region {j} alone")
        a, b, d = (host(x) for x in _grads(parts[i][0], parts[i][1], [0, len(parts[i][1])], [rho[j]], q, c, mode))
        want_v[nv[i]:nv[i + 1]], want_r[j], want_q = a, b[0], want_q + d
    assert maxrel(gq, want_q) < tol and maxrel(gr, want_r) < tol and maxrel(gv, want_v) < tol


@pytest.mark.parametrize("n,sub", [(200, 0), (40, 3)])  # one split each; 768 faces each
def test_time_of_the_sums(gpu, n, sub):
    v, t, off = _boxes(n, sub)
    rng = np.random.default_rng(2)
    q = dev(mg.q_random_ball(200, 0.5, rng))
    c = dev(rng.normal(size=200) + 0j)
    us = {}
    for kernel, kw in (("regions_finish_kernel", dict(need_verts=False, need_q=False)), ("dq_finish_kernel", {})):
        run = lambda: _grads(v, t, off, np.ones(n), q, c, "fp32c", **kw)  # noqa: B023,E731
        step(f"{kernel} of {n} regions")
        run()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            for _ in range(5):
                run()
            torch.cuda.synchronize()
        us[kernel] = min(e.device_time for e in p.events() if kernel in e.name)
    print(us)
    assert us["dq_finish_kernel"] < 1.8 * us["regions_finish_kernel"], us
