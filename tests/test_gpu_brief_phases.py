"""The binary64 adjoint's polynomials for short phases (|Q| rho <= 1.5, chosen per wavefront): lists whose phases are all
below, all above and on both sides of the limit, one mesh and a batch of two of different rho, against the oracle."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lat", [5, 16])  # 80 and 960 faces
@pytest.mark.parametrize("lo,hi", [(0.3, 1.45), (1.55, 2.9), (0.3, 2.9), (1.4, 4.0)])
def test_brief_phases(gpu, n_lat, lo, hi):
    v, t = mg.ellipsoid_uv([1.3, 1.0, 0.8], n_lat, centre=(0.2, -0.1, 0.3))
    rho = np.linalg.norm(v[t] - v[t].mean(axis=1, keepdims=True), axis=2).max()
    rng = np.random.default_rng(n_lat)
    for nq in (1, 200, 1500):
        q = rng.normal(size=(nq, 3))
        q *= (rng.uniform(lo, hi, size=nq) / rho / np.linalg.norm(q, axis=1))[:, None]
        c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
        A, B = dev(v), dev(t, torch.int32)
        want = O.grad3d(v, t, q, c)
        step(f"{len(t)} faces, {nq} Q, phases {lo} to {hi}")
        assert nrel(host(pft.backward_3d(A, B, dev(q), dev(c), mode="fp64")), want) < 1e-10
        half = O.grad3d(0.5 * v, t, q, c)
        got = host(pft.batch_backward(dev(np.r_[v, 0.5 * v]), dev(np.r_[t, t], torch.int32), dev(np.r_[q, q]),
                                      [0, len(v), 2 * len(v)], [0, len(t), 2 * len(t)], [0, nq, 2 * nq],
                                      dev(np.r_[c, c]), mode="fp64"))
        assert nrel(got[:len(v)], want) < 1e-10 and nrel(got[len(v):], half) < 1e-10
