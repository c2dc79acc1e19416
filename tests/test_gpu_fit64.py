"""The binary64 forms around the edge of their fitted phase range (largest centred vertex phase 3 rad), far beyond
it and at origin phases beyond 2^28 rad: forward, vertex adjoint and grad_Q against the oracle, at face counts
around the LDS tiles and Q counts around the cuts of small calls."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu

TOL_ADJOINT = 1e-10  # the binary64 adjoint's bar


def _mesh(nf):
    if nf == 12:
        return mg.box(1.0, 1.2, 0.8, origin=(-0.5, -0.6, -0.4))
    return mg.icosphere({80: 1, 320: 2}[nf], 1.0)


@pytest.mark.parametrize("nf", [12, 80, 320])
@pytest.mark.parametrize("phase", [0.05, 2.95, 3.1, 9.0, 60.0])
def test_binary64_across_the_fitted_range(gpu, nf, phase):
    v, t = _mesh(nf)
    v = v + np.array([0.2, -0.1, 0.3])
    g = v[t].mean(axis=1)
    rho = np.sqrt(((v[t] - g[:, None]) ** 2).sum(axis=2)).max()
    rng = np.random.default_rng(nf)
    for nq in (1, 63, 129, 600):
        q = mg.q_random_ball(nq, phase / rho, rng)
        if nq > 100:
            q[:20, :2] = 0.0  # along an axis (a face normal of the box)
        c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
        V, T, Q = dev(v), dev(t, torch.int32), dev(q)
        step(f"binary64 fitted range: {nf} faces, {nq} Q, phases to {phase}")
        assert nrel(host(pft.forward_3d(V, T, Q, mode="fp64")), O.ft3d(v, t, q)) < TOL_FP64
        step("binary64 fitted range: adjoint")
        assert nrel(host(pft.backward_3d(V, T, Q, dev(c), mode="fp64")), O.grad3d(v, t, q, c)) < TOL_ADJOINT
        step("binary64 fitted range: grad_Q")
        gq = pft.backward_3d_regions(V, T, [0, nf], dev(np.ones(1)), Q, dev(c), mode="fp64", need_verts=False,
                                     need_rho=False)[2]
        want = np.real(np.conj(c)[:, None] * O.ft3d_dq(v, t, q))
        assert nrel(host(gq), want) < TOL_ADJOINT


def test_origin_phases_beyond_the_reduction(gpu):
    """Two boxes 2e9 apart: origin phases up to 1e9 rad (the library sine there), each known to about 2^-53 times
    itself, 1e-7; the sum of two such terms and the oracle's own rounding stay below 2e-6."""
    v0, t0 = mg.box(1.0, 1.2, 0.8)
    v = np.concatenate([v0 - 1e9, v0 + 1e9])
    t = np.concatenate([t0, t0 + len(v0)]).astype(np.int32)
    rng = np.random.default_rng(4)
    q = mg.q_random_ball(200, 1.0, rng)
    c = rng.normal(size=200) + 1j * rng.normal(size=200)
    V, T, Q = dev(v), dev(t, torch.int32), dev(q)
    step("origin phases beyond 2^28")
    assert nrel(host(pft.forward_3d(V, T, Q, mode="fp64")), O.ft3d(v, t, q)) < 2e-6
    assert nrel(host(pft.backward_3d(V, T, Q, dev(c), mode="fp64")), O.grad3d(v, t, q, c)) < 2e-6
