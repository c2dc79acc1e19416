"""Zero-area faces (a repeated index, corners on one line) whose vertices differ contribute nothing to any gradient,
also where their centred phases lie beyond the fitted range (3 rad): every gradient equals that of the mesh without them,
in both forms. Faces and Q of both adjoint instances (small and full blocks), single, loss, regions and batch.

The faces' own terms are the same numbers with and without the extra faces; only the grouping of sums changes, so the
bound is a few hundred roundings of the largest entry: 1e-13 in binary64, 2e-6 in FP32C."""
import numpy as np
import pytest
import torch

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, host, maxrel, step

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-13, "fp32c": 2e-6}


def _mesh(level):
    """A closed mesh with three more vertices on a line parallel to x (exactly collinear), and the zero-area faces."""
    v, t = mg.icosphere(level, 1.0)
    n = len(v)
    v = np.concatenate([v, [[-0.5, 0.25, 0.125], [0.25, 0.25, 0.125], [0.75, 0.25, 0.125]]])
    zero = np.array([[0, 1, 1], [5, 2, 5], [7, 7, 3], [n, n + 1, n + 2], [n + 2, n, n + 1]], dtype=t.dtype)
    return v, t, zero


def _q(nq, phase, seed):
    """|Q| that gives the longest zero-area face (about 1.2 across, 0.66 to its centroid) the stated phase."""
    q = mg.q_random_ball(nq, 1.0, np.random.default_rng(seed))
    q /= np.linalg.norm(q, axis=1)[:, None]
    return q * (phase / 0.66)


CASES = [(1, 300, 5.0), (1, 300, 60.0), (3, 70000, 5.0), (3, 70000, 60.0)]  # small instance, full blocks


@pytest.mark.parametrize("mode", ["fp64", "fp32c"])
@pytest.mark.parametrize("level,nq,phase", CASES)
def test_single_mesh(gpu, mode, level, nq, phase):
    v, t, zero = _mesh(level)
    both = np.concatenate([t, zero])
    q = _q(nq, phase, 1)
    rng = np.random.default_rng(2)
    c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
    tgt = rng.random(nq)
    step(f"zero-area adjoint {mode} level {level}, {nq} Q, {phase} rad")
    got, want = (host(pft.backward_3d(dev(v), dev(x, torch.int32), dev(q), dev(c), mode=mode)) for x in (both, t))
    assert np.isfinite(got).all() and maxrel(got, want) < TOL[mode]
    step("zero-area loss")
    (lg, gg), (lw, gw) = (pft.intensity_loss_3d(dev(v), dev(x, torch.int32), dev(q), dev(tgt), mode=mode)
                          for x in (both, t))
    assert np.isfinite(host(gg)).all() and maxrel(host(gg), host(gw)) < 1e2 * TOL[mode]  # F^2 of cancelling sums
    assert maxrel(host(lg), host(lw)) < 1e2 * TOL[mode]


@pytest.mark.parametrize("mode", ["fp64", "fp32c"])
@pytest.mark.parametrize("level,nq,phase", CASES)
def test_regions(gpu, mode, level, nq, phase):
    v, t, zero = _mesh(level)
    inner = t.copy()
    v2 = np.concatenate([v, 0.5 * v])
    n = len(v)
    q = _q(nq, phase, 3)
    rng = np.random.default_rng(4)
    c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
    rho = dev(np.array([1.0, -0.7]))
    out = []
    for z in (zero, zero[:0]):
        parts = [np.concatenate([t, z]), np.concatenate([inner + n, z + n])]
        off = [0, len(parts[0]), len(parts[0]) + len(parts[1])]
        step(f"zero-area regions {mode} level {level}, {nq} Q, {phase} rad, {off[-1]} faces")
        out.append([host(x) for x in pft.backward_3d_regions(dev(v2), dev(np.concatenate(parts), torch.int32), off, rho,
                                                             dev(q), dev(c), mode=mode)])
    for got, want in zip(*out):
        assert np.isfinite(got).all() and maxrel(got, want) < 4 * TOL[mode]


@pytest.mark.parametrize("mode", ["fp64", "fp32c"])
def test_batch(gpu, mode):
    v, t, zero = _mesh(2)
    q = np.concatenate([_q(900, 5.0, 5), _q(2000, 60.0, 6)])
    c = np.random.default_rng(7).normal(size=(len(q), 2)) @ np.array([1.0, 1j])
    out = []
    for z in (zero, zero[:0]):
        one = np.concatenate([t, z])
        step(f"zero-area batch {mode}, {len(one)} faces a mesh")
        out.append(host(pft.batch_backward(dev(np.concatenate([v, v])), dev(np.concatenate([one, one]), torch.int32), dev(q),
                                           [0, len(v), 2 * len(v)], [0, len(one), 2 * len(one)], [0, 900, 2900],
                                           dev(c), mode=mode)))
    assert np.isfinite(out[0]).all() and maxrel(*out) < TOL[mode]
