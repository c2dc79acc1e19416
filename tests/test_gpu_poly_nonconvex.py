"""FP32C polygon faces of extreme non-convexity through their fan triangles, which then cancel: prisms over thin chevrons,
stars and combs (sides as triangles where that takes the caps of many edges through the triangle form). The bound is
that of binary32 terms summed over the fan: the face's terms T are each within 16 roundings, and within 4 |Q| rho more for
their phases (three products and two sums each), of at most |Q.N| / 2."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import dev, host, step

pytestmark = pytest.mark.gpu


def _star(points, inner):
    k = np.arange(2 * points)
    r = np.where(k % 2 == 0, 50.0, inner)
    return np.c_[r * np.cos(np.pi * k / points), r * np.sin(np.pi * k / points)]


def _comb(teeth):
    s, p = 60.0 / teeth, [(0.0, 0.0), (60.0, 0.0)]
    for k in range(teeth):
        x = 60.0 - k * s
        p += [(x, 43.0), (x - 0.45 * s, 43.0), (x - 0.45 * s, 3.0), (x - s, 3.0)]
    return np.array(p)


def _prism(poly, triangles):
    n = len(poly)
    v = np.concatenate([np.c_[poly, np.full(n, -15.0)], np.c_[poly, np.full(n, 15.0)]])
    f = [list(range(n))[::-1], list(range(n, 2 * n))]
    for i in range(n):
        j = (i + 1) % n
        f += [[i, j, n + j], [i, n + j, n + i]] if triangles else [[i, j, n + j, n + i]]
    return v - v.mean(axis=0), f


SHAPES = {"chevron": (np.array([(0.0, 0.0), (50.0, 25.0), (0.0, 50.0), (49.0, 25.0)]), False),
          "star": (_star(5, 4.0), False), "comb5": (_comb(5), True), "comb60": (_comb(60), True),
          "star60": (_star(60, 20.0), True)}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_cancelling_fans(gpu, name):
    poly, triangles = SHAPES[name]
    v, f = _prism(poly, triangles)
    rng = np.random.default_rng(len(poly))
    q = rng.normal(size=(400, 3))
    q *= (np.exp(rng.uniform(np.log(0.02), np.log(1.0), size=400)) / np.linalg.norm(q, axis=1))[:, None]
    q[:200, :2] *= 0.02  # nearly along the caps' normal
    tri = np.array([[p[0], p[k], p[k + 1]] for p in f for k in range(1, len(p) - 1)])
    a, b, c = v[tri[:, 0]], v[tri[:, 1]], v[tri[:, 2]]
    N = np.cross(b - a, c - a)
    rho = np.linalg.norm(np.stack([a, b, c]) - (a + b + c) / 3.0, axis=2).max()
    qn = np.linalg.norm(q, axis=1)
    scale = 0.5 * np.abs(q @ N.T).sum(axis=1) / qn ** 2
    step(f"prism over a {name} of {len(poly)} edges, {len(f)} faces")
    got = host(pft.forward_3d_poly(dev(v), f, dev(q), mode="fp32c"))
    err = np.abs(got - O.ft3d_poly(v, f, q))
    print("largest error over its bound", (err / ((16.0 + 4.0 * qn * rho) * 2.0 ** -24 * scale)).max())
    assert (err <= (16.0 + 4.0 * qn * rho) * 2.0 ** -24 * scale).all()
