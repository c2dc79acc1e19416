"""Batches about the list length (64 Q, a wavefront) up to which the Q order is left out: it would change no wavefront's Q.
Values against the meshes alone, non-finite and empty lists among them; and no sort where the longest list has 64 Q."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, host, maxrel, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest", [1, 64, 65])
@pytest.mark.parametrize("mode,tol", [("fp64", 1e-12), ("fp32c", 2e-5)])
def test_short_lists(gpu, longest, mode, tol):
    rng = np.random.default_rng(longest)
    n = 8192 if longest == 1 else 200  # at least 8 192 Q in all: where longer lists are sorted
    v, t = mg.box(3.0, 4.0, 5.0)
    qs = [mg.q_random_ball(longest, 0.8, rng) for _ in range(n)]
    if longest > 1:
        qs[3], qs[n - 1] = qs[3][:0], qs[n - 1][:7]
        qs[5][2, 1] = np.nan
    q, off = np.concatenate(qs), np.cumsum([0] + [len(x) for x in qs])
    assert len(q) >= 8192
    shift = rng.uniform(-1.0, 1.0, (n, 1, 3))
    V, T = dev((v + shift).reshape(-1, 3)), dev(np.tile(t, (n, 1)), torch.int32)
    vo, to = np.arange(n + 1) * len(v), np.arange(n + 1) * len(t)
    c = rng.normal(size=len(q)) + 1j * rng.normal(size=len(q))
    step(f"batch of {n} lists of up to {longest} Q, {mode}")
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        F = host(pft.batch_forward(V, T, dev(q), vo, to, off, mode=mode))
        G = host(pft.batch_backward(V, T, dev(q), vo, to, off, dev(c), mode=mode)).reshape(n, -1, 3)
    assert any("sort_scatter_kernel" in e.name for e in p.events()) == (longest > 64)
    for i in (0, 3, 5, n // 2, n - 1) if longest > 1 else (0, n - 1):
        A, qi = dev(v + shift[i]), dev(q[off[i]:off[i + 1]])
        B = dev(t, torch.int32)
        Fi = F[off[i]:off[i + 1]]
        if len(qi) == 0:
            assert not G[i].any()
            continue
        f = host(pft.forward_3d(A, B, qi, mode=mode))
        ok = np.isfinite(q[off[i]:off[i + 1]]).all(axis=1)
        assert np.isnan(Fi[~ok]).all() and nrel(Fi[ok], f[ok]) < tol
        g = host(pft.backward_3d(A, B, qi, dev(c[off[i]:off[i + 1]]), mode=mode))
        if ok.all():
            assert maxrel(G[i], g) < tol * 10
        else:
            assert np.array_equal(np.isnan(G[i]), np.isnan(g))
