"""The fitted polynomials of csrc/face_poly.h: the face integral J and the barycentric moments Y_k they give
against the converged series, on triangles up to the edge of the fitted phase range."""
import math
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2104_08309_amd", "csrc")


def _fits():
    with open(os.path.join(CSRC, "face_poly.h")) as fh:
        src = fh.read()
    out = {}
    for m in re.finditer(r"struct (FaceFit\w+) \{\n  static constexpr double M = ([0-9.]+);\n(.*?)\n\};", src, re.S):
        tab = {}
        for t in re.finditer(r"struct ([A-Za-z]+)(\d) \{ static constexpr \w+ c\[(\d+)\] = \{([^}]*)\};", m.group(3)):
            c = np.array([float(x.strip().rstrip("f")) for x in t.group(4).split(",")])
            assert len(c) == int(t.group(3))
            tab.setdefault(t.group(1), []).append(c)
        out[m.group(1)] = (float(m.group(2)), tab)
    return out


def _series(d, nmax=60):
    """J and Y_k by the recursions in n (independent of the symmetric form)."""
    d0, d1, d2 = d
    e2, e3 = d0 * d1 + d1 * d2 + d2 * d0, d0 * d1 * d2
    H = [np.ones_like(d0), np.zeros_like(d0), -e2]
    for n in range(3, nmax + 1):
        H.append(-e2 * H[n - 2] + e3 * H[n - 3])
    J = sum((1j ** n) * H[n] / math.factorial(n + 2) for n in range(nmax + 1))
    Y = []
    for k in range(3):
        a = np.ones_like(d0)
        y = a / 6.0 + 0j
        for n in range(1, nmax + 1):
            a = H[n] + d[k] * a
            y = y + (1j ** n) * a / math.factorial(n + 3)
        Y.append(y)
    return J, Y


@pytest.mark.parametrize("name,tol_j,tol_y", [("FaceFit32", 4e-8, None), ("FaceFit32M", 4e-8, 4e-8),
                                              ("FaceFit64", 4e-16, 4e-16), ("FaceFit64S", 4e-16, 4e-16)])
def test_face_fit(name, tol_j, tol_y):
    """Tolerances: the fits' own errors (at most 2.5e-8 for J and 2.2e-8 for a moment's parts in binary32, rounded
    coefficients beside them; below 1e-16 in binary64, where a few roundings of values near 1/2 remain)."""
    M, tab = _fits()[name]
    scale = 4.0 * math.pi if name == "FaceFit32" else 1.0
    rng = np.random.default_rng(9)
    d = rng.normal(size=(3, 4000))
    d -= d.mean(axis=0)
    d *= M * np.where(np.arange(4000) % 4 == 0, 1.0, rng.random(4000)) / np.abs(d).max(axis=0)
    d[2] = -d[0] - d[1]  # exactly centred
    x = d / scale
    p, E = x[0] ** 2 + x[0] * x[1] + x[1] ** 2, x[0] * x[1] * (x[0] + x[1])
    f = {k: sum(np.polyval(c[::-1], p) * (E * E) ** i for i, c in enumerate(cs)) for k, cs in tab.items()}
    J = f["A"] + 1j * E * f["B"]
    if tol_y is None:
        assert np.max(np.abs(J - _series(d)[0])) < tol_j
        return
    beta, gamma = 1j * f["bi"] + E * f["br"], f["gr"] + 1j * E * f["gi"]
    J0, Y0 = _series(d)
    assert np.max(np.abs(J - J0)) < tol_j
    alpha = (J - 2.0 * p * scale ** 2 * gamma) / 3.0
    for k in range(3):
        assert np.max(np.abs(alpha + beta * d[k] + gamma * d[k] ** 2 - Y0[k])) < tol_y * max(1.0, M), k


def test_face_fit_at_zero():
    """A face without extent has J = 1/2 exactly (every small face is scaled by it)."""
    for _, tab in _fits().values():
        assert tab["A"][0][0] == 0.5
