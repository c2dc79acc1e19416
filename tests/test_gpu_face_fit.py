"""The FP32C forward around the edge of its fitted phase range (largest centred vertex phase 3.6 rad): small
phases, ranges that straddle the edge inside one wavefront and one face list, and phases far beyond it, at face
counts around the LDS tile and Q counts around the cuts of small calls; in both face orders, against the oracle."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, dev, host, nrel, step

pytestmark = pytest.mark.gpu


def _mesh(nf):
    if nf == 12:
        return mg.box(1.0, 1.2, 0.8, origin=(-0.5, -0.6, -0.4))
    return mg.icosphere({80: 1, 320: 2, 1280: 3}[nf], 1.0)


@pytest.mark.parametrize("nf", [12, 80, 320, 1280])
@pytest.mark.parametrize("phase", [0.05, 3.55, 3.7, 9.0, 60.0])
def test_forward_across_the_fitted_range(gpu, nf, phase):
    v, t = _mesh(nf)
    v = v + np.array([0.2, -0.1, 0.3])
    g = v[t].mean(axis=1)
    rho = np.sqrt(((v[t] - g[:, None]) ** 2).sum(axis=2)).max()
    rng = np.random.default_rng(nf)
    for nq in (1, 63, 129, 700):
        q = mg.q_random_ball(nq, phase / rho, rng)
        if nq > 100:
            q[:20, :2] = 0.0  # along an axis (a face normal of the box)
        q32, v32 = q.astype(np.float32).astype(np.float64), v.astype(np.float32).astype(np.float64)
        want = O.ft3d(v32, t, q32)
        T = dev(t, torch.int32)
        order = tuple(dev(x) for x in pft.strip_order(t))
        for name, o in (("list order", None), ("edge-sharing order", order)):
            step(f"fitted range {name}: {nf} faces, {nq} Q, phases to {phase}")
            got = host(pft.forward_3d(dev(v, torch.float32), T, dev(q, torch.float32), mode="fp32c", order=o))
            assert nrel(got, want) < TOL_FP32C, (name, nq)


def test_value_does_not_depend_on_the_other_q(gpu):
    """Q on both sides of the range's edge in one wavefront: a permuted list gives bitwise the same values."""
    v, t = mg.icosphere(2, 1.0)
    rng = np.random.default_rng(3)
    q = np.concatenate([mg.q_random_ball(500, 5.0, rng), mg.q_random_ball(500, 40.0, rng)])
    perm = rng.permutation(len(q))
    V, T = dev(v, torch.float32), dev(t, torch.int32)
    for o in (None, tuple(dev(x) for x in pft.strip_order(t))):
        step("fitted range: permuted list")
        a = host(pft.forward_3d(V, T, dev(q, torch.float32), mode="fp32c", order=o))
        b = host(pft.forward_3d(V, T, dev(q[perm], torch.float32), mode="fp32c", order=o))
        assert np.array_equal(b.view(np.uint8), a[perm].view(np.uint8))
