"""Polygon faces through their fan triangles and through the polygon kernel: prisms whose face sizes lie on both sides
of the rule that picks one, phases below and beyond the fitted range, non-convex faces, empty faces between full ones
(a chain of fan triangles must not link across them), in both forms against the oracle."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, TOL_FP64, dev, host, nrel, special_q, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [3, 4, 5, 6, 7, 12, 40])
def test_prisms(gpu, nu):
    ang = 2.0 * np.pi * np.arange(nu) / nu
    rad = np.where(np.arange(nu) % 2 == 0, 1.0, 0.7 if nu > 5 else 1.0)  # non-convex from 6 up
    v, f = mg.prism_polygon(np.c_[rad * np.cos(ang), rad * np.sin(ang)] + 0.1, 1.4, -0.3)
    rng = np.random.default_rng(nu)
    for qmax in (0.5, 6.0, 45.0):
        q = np.concatenate([mg.q_random_ball(300, qmax, rng), special_q(qmax)])
        want = O.ft3d_poly(v, f, q)
        bad = f[:1] + [[0, 1, 10 ** 6]] + f[1:3] + [[0, 0, 0]] + f[3:]
        for mode, tol in (("fp64", TOL_FP64), ("fp32c", TOL_FP32C)):
            for name, faces in (("plain", f), ("with empty faces", bad)):
                step(f"prism of {nu}-gons {mode} {name} to |Q| = {qmax}")
                got = host(pft.forward_3d_poly(dev(v), faces, dev(q), mode=mode))
                assert nrel(got, want) < tol, (mode, name, qmax)
