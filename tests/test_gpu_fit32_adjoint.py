"""The FP32C adjoint and grad_Q around the edge of the fitted phase range of their moments (largest centred vertex
phase 3 rad), far beyond it, and at origin phases beyond 2^19 turns, against the oracle."""
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
    return mg.icosphere({80: 1, 320: 2}[nf], 1.0)


@pytest.mark.parametrize("nf", [12, 80, 320])
@pytest.mark.parametrize("phase", [0.3, 2.95, 3.1, 9.0, 60.0])
def test_adjoint_across_the_fitted_range(gpu, nf, phase):
    v, t = _mesh(nf)
    v = v + np.array([0.2, -0.1, 0.3])
    g = v[t].mean(axis=1)
    rho = np.sqrt(((v[t] - g[:, None]) ** 2).sum(axis=2)).max()
    rng = np.random.default_rng(nf)
    for nq in (1, 257, 800):
        q = mg.q_random_ball(nq, phase / rho, rng)
        q[:nq // 8, :2] = 0.0  # along an axis (a face normal of the box)
        c = (rng.normal(size=nq) + 1j * rng.normal(size=nq)).astype(np.complex64)
        V, T, Q = dev(v), dev(t, torch.int32), dev(q)
        step(f"FP32C moments: {nf} faces, {nq} Q, phases to {phase}")
        got = host(pft.backward_3d(V, T, Q, dev(c), mode="fp32c"))
        assert nrel(got, O.grad3d(v, t, q, c)) < TOL_FP32C
        step("FP32C moments: grad_Q")
        gq = pft.backward_3d_regions(V, T, [0, nf], dev(np.ones(1)), Q, dev(c), mode="fp32c", need_verts=False,
                                     need_rho=False)[2]
        want = np.real(np.conj(c)[:, None] * O.ft3d_dq(v, t, q))
        assert nrel(host(gq), want) < TOL_FP32C


def test_origin_phases_beyond_the_fixed_point_range(gpu):
    """Two boxes 2e7 apart: origin phases up to 1e7 rad, 1.6e6 turns (the plain reduction there)."""
    v0, t0 = mg.box(1.0, 1.2, 0.8)
    v = np.concatenate([v0 - 6e6, v0 + 6e6])
    t = np.concatenate([t0, t0 + len(v0)]).astype(np.int32)
    rng = np.random.default_rng(4)
    q = mg.q_random_ball(200, 1.0, rng) + np.array([1.0, 0.0, 0.0])
    c = (rng.normal(size=200) + 1j * rng.normal(size=200)).astype(np.complex64)
    V, T, Q = dev(v), dev(t, torch.int32), dev(q)
    step("FP32C adjoint: origin phases beyond 2^19 turns")
    assert nrel(host(pft.backward_3d(V, T, Q, dev(c), mode="fp32c")), O.grad3d(v, t, q, c)) < TOL_FP32C
