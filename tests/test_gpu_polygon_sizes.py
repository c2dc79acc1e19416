"""The 2D transform on both sides of its one-launch limit (one contour of at most 256 vertices), against the oracle:
edge phases below and above pi/4, Q = 0 and the small-|Q| fan, phases beyond the range of the polynomial sines."""
import numpy as np
import pytest

import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu


def contour(nv):
    a = 2.0 * np.pi * np.arange(nv) / nv
    r = 1.0 + 0.3 * np.cos(3 * a)
    return np.c_[r * np.cos(a) + 0.4, 0.7 * r * np.sin(a) - 0.2]


@pytest.mark.parametrize("nv", [3, 5, 63, 64, 65, 255, 256, 257, 600])
@pytest.mark.parametrize("nq", [1, 31, 33, 1000])
def test_polygon_sizes(gpu, nv, nq):
    v = contour(nv)
    rng = np.random.default_rng(nv + nq)
    for qmax in (0.01, 2.0, 40.0, 400.0):
        q = rng.uniform(-qmax, qmax, size=(nq, 2))
        q[nq // 2:nq // 2 + 1] = 0.0
        want = O.ft2d(v, q)
        step(f"{nv}-gon, {nq} Q to {qmax}")
        assert nrel(host(pft.forward_2d(dev(v), dev(q))), want) < TOL_FP64
        one = host(pft.forward_2d(dev(v), dev(q), contour_offsets=[0, nv]))
        assert nrel(one, want) < TOL_FP64
        if nv > 5:  # the same polygon cut into two contours along a chord: the general launches
            cut = np.concatenate([v[:nv // 2 + 1], v[nv // 2:], v[:1]])
            two = host(pft.forward_2d(dev(cut), dev(q), contour_offsets=[0, nv // 2 + 1, nv + 2]))
            assert nrel(two, want) < TOL_FP64


@pytest.mark.parametrize("nv", [4, 7, 256, 257])
@pytest.mark.parametrize("nq", [131071, 131072, 131201])
def test_long_lists(gpu, nv, nq):
    """Both sides of the rule on the edge groups; the oracle on a sample with the last Q."""
    v = contour(nv)
    q = np.random.default_rng(nq).uniform(-30.0, 30.0, size=(nq, 2))
    q[5] = 0.0
    step(f"{nv}-gon, {nq} Q")
    got = host(pft.forward_2d(dev(v), dev(q)))
    sel = np.concatenate([np.arange(8), np.arange(nq - 300, nq)])
    assert nrel(got[sel], O.ft2d(v, q[sel])) < TOL_FP64


@pytest.mark.parametrize("nv", [4, 300])
def test_wide_phases(gpu, nv):
    """|Q| R on both sides of 2^28 within a wavefront; the phases themselves carry 1e9 * 2^-52 * a few."""
    v = contour(nv)
    rng = np.random.default_rng(nv)
    q = rng.uniform(-1.0, 1.0, size=(96, 2)) * np.where(np.arange(96) % 3 == 0, 8e8, 1e6)[:, None]
    q[7] = [np.inf, 1.0]
    q[9] = [np.nan, 1.0]
    step(f"{nv}-gon, wide phases")
    got = host(pft.forward_2d(dev(v), dev(q)))
    ok = np.isfinite(q).all(axis=1)
    assert not np.isfinite(got[~ok]).any()
    q2 = (q[ok] ** 2).sum(axis=1)  # F |Q|^2 / |Q| is of the order of the perimeter: compare at that scale
    err = np.abs(got[ok] - O.ft2d(v, q[ok])) * np.sqrt(q2)
    assert err.max() < 1e-5
