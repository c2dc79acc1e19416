"""The orientation average on both sides of the rule that sorts its Q list (fewer than 256 directions), with shuffled
magnitudes (0 and repeated ones among them) and directions, against the average of the transform's own intensities
and the oracle at sampled magnitudes."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndir", [255, 256, 300])
@pytest.mark.parametrize("mode,tol", [("fp64", TOL_FP64), ("fp32c", TOL_FP32C)])
def test_orient_order(gpu, ndir, mode, tol):
    v, t = mg.ellipsoid_uv([1.3, 1.0, 0.8], 12, centre=(0.2, -0.1, 0.3))
    rng = np.random.default_rng(ndir)
    d = rng.normal(size=(ndir, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    w = rng.random(ndir) / ndir
    qa = rng.permutation(np.concatenate([np.linspace(0.0, 9.0, 60), [9.0, 0.0, 1e-3]]))
    A, B = dev(v), dev(t, torch.int32)
    step(f"{len(qa)} magnitudes x {ndir} directions {mode}")
    got = host(pft.orientation_average(A, B, dev(qa), dev(d), dev(w), mode=mode))
    q = (qa[:, None, None] * d[None]).reshape(-1, 3)
    F = host(pft.forward_3d(A, B, dev(q), mode=mode, intensity=True)[1]).astype(np.float64).reshape(len(qa), ndir)
    assert nrel(got, F @ w) < tol
    sel = [0, 7, 31, 62]
    assert nrel(got[sel], O.orientation_average(v, t, qa[sel], d, w)) < 4 * tol  # |F|^2: twice the transform's, summed
