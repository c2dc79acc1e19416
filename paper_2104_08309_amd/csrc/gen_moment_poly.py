"""Writes moment_poly.h: polynomials of exp(ix) for a triangle's face integral and barycentric
moments at small centred vertex phases in binary32. The polygon kernel uses FacePoly; the bucketed
MomentPoly are kept as checked tables that no kernel uses (the adjoint's moments come from the
symmetric fits of gen_face_poly.py).

The face integral of exp(iQ.x) over a triangle, normalised by twice its area, and the
moments of the barycentric coordinates are averages over the standard simplex of
exp(i phi(lambda)) and lambda_k exp(i phi(lambda)), with phi(lambda) = sum_j lambda_j d_j
linear in the barycentric coordinates (d_j the centred vertex phases, sum d_j = 0). A
polynomial q(x) = sum_n a_n i^n x^n turns them into finite sums, since the simplex
averages of phi^n are complete homogeneous symmetric polynomials:

    J   = sum_n i^n a_n n! h_n(d0, d1, d2)      / (n+2)!
    Y_k = sum_n i^n a_n n! h_n(d0, d1, d2, d_k) / (n+3)!

and because phi(lambda) stays in [-m, m] (m = max |d_j|, a convex combination), a q with
|q(x) - exp(ix)| <= eps on [-M, M], M >= m, puts J within eps/2 and Y_k within eps/6 of
the exact moments (the simplex has area 1/2, each moment weight integrates to 1/6). The
Taylor polynomial (a_n = 1/n!) needs about e M + log(1/eps) terms; Chebyshev
interpolation of cos and sin on [-M, M] (at the Chebyshev points of the first kind,
mapped to [-M, M]) needs fewer, its error being about 2 (M/2)^(N+1) / (N+1)! against
M^(N+1) / (N+1)! for Taylor. One polynomial per phase bucket M.

Run from this directory: python gen_moment_poly.py > moment_poly.h
"""
import math

import numpy as np
from numpy.polynomial import chebyshev as C

# M in radians, exact in binary32, each just below the range where the next degree is needed at EPS;
# the last one is the adjoint's series/edge switch.
BUCKETS = (0.6875, 1.03125, 1.4375, 1.875, 2.34375, 2.84375, 3.0)
# Target |q(x) - exp(ix)| on [-M, M] (complex modulus): J within 4e-7 and Y_k within 1.3e-7, the size of
# the truncation error of the Taylor form stopped at m^n / n! < 1e-6.
EPS = 8.0e-7
# The forward's near-degenerate pairs (Q nearly along the face normal) need only the face integral J, at
# small phases; one polynomial on [-FACE_M, FACE_M] with J within FACE_EPS/2 (a lane beyond FACE_M keeps the
# binary64 series).
FACE_M = 0.5
FACE_EPS = 2.0e-7
GRID = 20001


def fit(fun, M, deg, parity):
    """Chebyshev interpolant of fun(M t) on t in [-1, 1] of degree deg, as monomial
    coefficients in x = M t (coefficients of the other parity set to zero)."""
    ct = C.chebinterpolate(lambda t: fun(M * t), deg)
    pt = C.cheb2poly(ct)
    px = np.array([pt[n] / M ** n for n in range(len(pt))])
    for n in range(len(px)):
        if n % 2 != parity:
            px[n] = 0.0
    return px


def max_err(px, fun, M):
    x = np.linspace(-M, M, GRID)
    return float(np.max(np.abs(np.polynomial.polynomial.polyval(x, px) - fun(x))))


def smallest(fun, M, parity, eps):
    for deg in range(parity, 40, 2):
        px = fit(fun, M, deg, parity)
        px32 = px.astype(np.float32).astype(np.float64)
        if max_err(px32, fun, M) <= eps:
            return deg, px
    raise RuntimeError("no degree below 40")


def bucket(M, eps_total=None):
    eps = (EPS if eps_total is None else eps_total) / math.sqrt(2.0)
    dc, pc = smallest(np.cos, M, 0, eps)
    ds, ps = smallest(np.sin, M, 1, eps)
    N = max(dc, ds)
    a = np.zeros(N + 1)
    for n in range(N + 1):
        # i^n a_n x^n: real part (-1)^(n/2) a_n for even n, imaginary (-1)^((n-1)/2) a_n for odd n
        sgn = (-1.0) ** (n // 2)
        src = pc if n % 2 == 0 else ps
        a[n] = sgn * src[n] if n < len(src) else 0.0
    cj = [a[n] * math.factorial(n) / math.factorial(n + 2) for n in range(N + 1)]
    cy = [a[n] * math.factorial(n) / math.factorial(n + 3) for n in range(N + 1)]
    x = np.linspace(-M, M, GRID)
    q = sum((1j ** n) * float(np.float32(a[n])) * x ** n for n in range(N + 1))
    err = float(np.max(np.abs(q - np.exp(1j * x))))
    return N, dc, ds, cj, cy, err


def main():
    out = []
    out.append("// Generated by gen_moment_poly.py (Chebyshev interpolation of cos and sin); do not edit.")
    out.append("// Polynomials q(x) = sum_n i^n a_n x^n of exp(ix) on [-M, M] for the binary32 barycentric")
    out.append("// moments: cj[n] = a_n n!/(n+2)! (face integral J), cy[n] = a_n n!/(n+3)! (moments Y_k).")
    out.append("// err = max |q(x) - exp(ix)| on [-M, M] with a_n rounded to binary32; J is then within err/2")
    out.append("// and Y_k within err/6 of the exact moments for every triangle with max |d_k| <= M.")
    out.append("// The polygon kernel uses FacePoly; no kernel uses the MomentPoly.")
    out.append("#pragma once")
    out.append("")
    out.append("namespace pft {")
    out.append("")
    for b, M in enumerate(BUCKETS):
        N, dc, ds, cj, cy, err = bucket(M)
        name = f"MomentPoly{b}"
        out.append(f"// M = {M}: cos to degree {dc}, sin to degree {ds}; err = {err:.2e}")
        out.append(f"struct {name} {{")
        out.append(f"  static constexpr float M = {M!r}f;")
        out.append(f"  static constexpr int N = {N};")
        out.append("  static constexpr float cj[N + 1] = {" + ", ".join(f"{float(np.float32(v))!r}f" for v in cj) + "};")
        out.append("  static constexpr float cy[N + 1] = {" + ", ".join(f"{float(np.float32(v))!r}f" for v in cy) + "};")
        out.append("};")
        out.append("")
    N, dc, ds, cj, cy, err = bucket(FACE_M, FACE_EPS)
    out.append(f"// Face integral only, M = {FACE_M}: cos to degree {dc}, sin to degree {ds}; err = {err:.2e}")
    out.append("struct FacePoly {")
    out.append(f"  static constexpr float M = {FACE_M!r}f;")
    out.append(f"  static constexpr int N = {N};")
    out.append("  static constexpr float cj[N + 1] = {" + ", ".join(f"{float(np.float32(v))!r}f" for v in cj) + "};")
    out.append("};")
    out.append("")
    out.append(f"constexpr int kMomentPolyBuckets = {len(BUCKETS)};")
    out.append(f"constexpr double kMomentPolyMaxPhase = {BUCKETS[-1]!r};")
    out.append(f"constexpr double kMomentPolyErr = {EPS!r};")
    out.append(f"constexpr double kFacePolyErr = {FACE_EPS!r};")
    out.append("")
    out.append("}  // namespace pft")
    print("\n".join(out))


if __name__ == "__main__":
    main()
