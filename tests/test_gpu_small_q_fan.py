"""The small-|Q| tetrahedron fans: 1, 8, 9, 64 and 300 small Q among others (one served at a time by its whole wavefront,
a face per lane, up to 8 of them; beyond that each by its own lane), on lists that end inside a Q tile, over face counts
about a wavefront and a tile, for the transform, grad_Q and batches, in both forms, against the oracle. A Q's transform
does not depend on its neighbours in the list."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lat", [3, 5, 11, 24])  # 24, 80, 440, 2 208 faces
@pytest.mark.parametrize("n_small", [1, 8, 9, 64, 300])
def test_fans(gpu, n_lat, n_small):
    v, t = mg.ellipsoid_uv([1.3, 1.0, 0.8], n_lat, centre=(0.2, -0.1, 0.3))
    rng = np.random.default_rng(n_lat + n_small)
    q = mg.q_random_ball(333, 6.0, rng)
    at = rng.permutation(333)[:n_small]
    q[at] = mg.q_random_ball(n_small, 0.01, rng)  # |Q| R < 0.02: within every form's fan
    q[at[0]] = 0.0
    F, dF, A, B = O.ft3d(v, t, q), O.ft3d_dq(v, t, q), dev(v), dev(t, torch.int32)
    for mode, tol in (("fp64", TOL_FP64), ("fp32c", TOL_FP32C)):
        step(f"{len(t)} faces, {n_small} small Q, {mode}")
        got = host(pft.forward_3d(A, B, dev(q), mode=mode))
        assert nrel(got, F) < tol
        assert nrel(got[at], F[at]) < tol
        one = host(pft.forward_3d(A, B, dev(q[at[:1]]), mode=mode))
        few = host(pft.forward_3d(A, B, dev(np.repeat(q[at[:1]], 70, axis=0)), mode=mode))
        assert np.array_equal(few, np.repeat(one, 70))
        c = rng.normal(size=333) + 1j * rng.normal(size=333)
        c = c if mode == "fp64" else c.astype(np.complex64)
        gq = pft.backward_3d_regions(A, B, [0, len(t)], dev(np.ones(1)), dev(q), dev(c), mode=mode, need_verts=False,
                                     need_rho=False)[2]
        assert nrel(host(gq), np.real(np.conj(c)[:, None] * dF)) < (1e-10 if mode == "fp64" else TOL_FP32C)
        vo, to, qo = [0, len(v), 2 * len(v)], [0, len(t), 2 * len(t)], [0, 300, 333]
        bt = host(pft.batch_forward(dev(np.r_[v, v]), dev(np.r_[t, t], torch.int32), dev(q), vo, to, qo, mode=mode))
        assert nrel(bt, F) < tol
