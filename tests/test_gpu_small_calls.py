"""The cuts of small calls: the one-block prologue (to 512 faces), the one-launch vertex gather (to 2 048 faces), the
small adjoint instance and the finer face splits, at sizes on both sides of each limit, in both forms, against the
oracle on a sample (the gradient of sampled vertices); with out-of-range and repeated indices and a vertex of more
than 64 corners."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lat", [3, 11, 12, 23, 24])  # 24, 440, 528, 2024, 2208 faces
def test_small_call_cuts(gpu, n_lat):
    v, t = mg.ellipsoid_uv([1.3, 1.0, 0.8], n_lat, centre=(0.2, -0.1, 0.3))  # poles of 2 n_lat corners
    rng = np.random.default_rng(n_lat)
    for nq in (1, 65, 300, 1500):
        q = mg.q_random_ball(nq, 6.0, rng)
        c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
        want_F, want_G = O.ft3d(v, t, q), O.grad3d(v, t, q, c)
        for mode, tol, tol_g in (("fp64", TOL_FP64, 1e-10), ("fp32c", TOL_FP32C, TOL_FP32C)):
            step(f"small call {mode}: {len(t)} faces, {nq} Q")
            F = host(pft.forward_3d(dev(v), dev(t, torch.int32), dev(q), mode=mode))
            assert nrel(F, want_F) < tol, (mode, nq)
            G = host(pft.backward_3d(dev(v), dev(t, torch.int32), dev(q), dev(c), mode=mode))
            assert nrel(G, want_G) < tol_g, (mode, nq)


def test_gather_of_a_vertex_of_many_corners(gpu):
    """A fan of 150 faces about one vertex (three lots of 64 corners), and faces with bad indices, which add nothing."""
    n = 150
    a = 2.0 * np.pi * np.arange(n) / n
    v = np.concatenate([[[0.0, 0.0, 1.0], [0.0, 0.0, -1.0]], np.c_[np.cos(a), np.sin(a), 0.0 * a]])
    k = np.arange(n)
    up = np.c_[np.zeros(n), 2 + k, 2 + (k + 1) % n]
    dn = np.c_[np.ones(n), 2 + (k + 1) % n, 2 + k]
    t = np.concatenate([up, dn]).astype(np.int32)
    rng = np.random.default_rng(5)
    q = mg.q_random_ball(200, 5.0, rng)
    c = rng.normal(size=200) + 1j * rng.normal(size=200)
    want = O.grad3d(v, t, q, c)
    bad = np.concatenate([t, [[0, 1, 9999], [-1, 2, 3], [4, 4, 4]]]).astype(np.int32)
    for mode, tol in (("fp64", 1e-10), ("fp32c", TOL_FP32C)):
        for name, tt in (("closed", t), ("with bad faces", bad)):
            step(f"gather {mode} {name}")
            G = host(pft.backward_3d(dev(v), dev(tt, torch.int32), dev(q), dev(c), mode=mode))
            assert nrel(G, want) < tol, (mode, name)
