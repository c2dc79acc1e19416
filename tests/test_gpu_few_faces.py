"""The FP32C forward of few faces, which writes F itself: face counts on both sides of its limits (16, and 32 from
2^18 Q), Q counts about its blocks of 256, |F|^2, Q = 0 and the small-|Q| fan, phases beyond the fixed-point
range and beyond the mode's, a caller's Q order (which must not change a value), against the oracle on a sample."""
import numpy as np
import pytest
import torch

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, dev, host, nrel, special_q, step

pytestmark = pytest.mark.gpu


def closed_mesh(nf):
    """A closed prism of 4 n - 4 faces over an n-gon (12 from n = 4, 36 from n = 10)."""
    n = nf // 4 + 1
    a = 2.0 * np.pi * np.arange(n) / n
    lo, hi = np.c_[np.cos(a), 0.8 * np.sin(a), 0.0 * a - 0.5], np.c_[np.cos(a), 0.8 * np.sin(a), 0.0 * a + 0.7]
    k, k1 = np.arange(n), (np.arange(n) + 1) % n
    i = np.arange(1, n - 1)
    t = np.concatenate([np.c_[k, k1, n + k1], np.c_[k, n + k1, n + k], np.c_[0 * i, i + 1, i],
                        np.c_[0 * i + n, n + i, n + i + 1]])
    assert len(t) == nf
    return np.concatenate([lo, hi]) + [0.3, -0.2, 0.1], t.astype(np.int32)


@pytest.mark.parametrize("nf", [8, 12, 16, 20, 32, 36])
@pytest.mark.parametrize("nq", [1, 255, 257, 9000, 65535, 262143, 262144, 524801])
def test_few_faces(gpu, nf, nq):
    v, t = closed_mesh(nf)
    rng = np.random.default_rng(nf + nq)
    rho = np.linalg.norm(v[t] - v[t].mean(axis=1, keepdims=True), axis=2).max()
    for qmax in (0.01, 0.4, 9.0, 70.0):  # 0.01: every Q through the fan
        step(f"{nf} faces, {nq} Q to |Q| = {qmax}")
        q = mg.q_random_ball(nq, qmax, rng)
        sp = special_q(qmax)[:max(nq - 1, 0)]
        q[nq - len(sp):] = sp
        Q = dev(q)
        out, inten = pft.forward_3d(dev(v), dev(t, torch.int32), Q, mode="fp32c", intensity=True)
        sel = np.unique(np.concatenate([np.arange(max(nq - 40, 0), nq), rng.integers(0, nq, 60)]))
        want = O.ft3d(v, t, q[sel])
        beyond = np.linalg.norm(q[sel], axis=1) * rho > 128.0  # the mode's documented range: NaN
        assert np.array_equal(np.isnan(host(out)[sel]), beyond) and np.array_equal(np.isnan(host(inten)[sel]), beyond)
        F, I, want = host(out)[sel][~beyond], host(inten)[sel][~beyond], want[~beyond]
        assert nrel(F, want) < TOL_FP32C
        assert np.abs(I - np.abs(want) ** 2).max() < 4 * TOL_FP32C * np.abs(want).max() ** 2
        ordered = pft.forward_3d(dev(v), dev(t, torch.int32), Q, mode="fp32c", q_order=pft.q_order(Q))
        assert np.array_equal(host(ordered), host(out), equal_nan=True)


def test_few_faces_wide_phases(gpu):
    """Two small tetrahedra so far apart that |Q| R lies on both sides of the fixed-point range (3.2e6 rad) within a
    wavefront, then phases beyond the mode's range and a NaN, which give NaN at their own Q only."""
    a = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
    f = np.array([[0, 2, 1], [0, 1, 3], [1, 2, 3], [0, 3, 2]])
    v = np.concatenate([a, a * [1, 0.7, 1.2] + [2.0e6, 1.0e6, 0.5e6]])
    t = np.concatenate([f, f + 4]).astype(np.int32)
    R = 0.5 * np.linalg.norm([2.0e6, 1.0e6, 0.5e6])
    rng = np.random.default_rng(3)
    q = rng.normal(size=(700, 3))
    q *= (rng.uniform(0.5, 4.5, size=700) / np.linalg.norm(q, axis=1))[:, None]
    qr = np.linalg.norm(q, axis=1) * R
    assert (qr < 3.1e6).any() and (qr > 3.3e6).any()
    step("two tetrahedra, |Q| R about 3.2e6")
    got = host(pft.forward_3d(dev(v), dev(t, torch.int32), dev(q), mode="fp32c"))
    assert nrel(got, O.ft3d(v, t, q)) < TOL_FP32C
    q[5] = [1e16, 0, 0]
    q[6] = [np.nan, 0, 0]
    step("beyond the mode's range")
    bad = host(pft.forward_3d(dev(v), dev(t, torch.int32), dev(q), mode="fp32c"))
    assert np.isnan(bad[[5, 6]]).all()
    assert np.array_equal(np.delete(bad, [5, 6]), np.delete(got, [5, 6]))
