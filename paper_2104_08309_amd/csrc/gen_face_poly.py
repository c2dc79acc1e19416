"""Writes face_poly.h: fitted polynomials for a triangle's face integral and barycentric moments.

With the centred vertex phases d_0 + d_1 + d_2 = 0 of a triangle, the face integral of exp(i phase)
normalised by twice the area and the moment of the barycentric coordinate of vertex k are

    J   = sum_n i^n h_n(d_0, d_1, d_2) / (n+2)!,      Y_k = sum_n i^n h_n(d_0, d_1, d_2, d_k) / (n+3)!,

h_n the complete homogeneous symmetric polynomials. J is symmetric in the d, so it is a function of
p = d_0^2 + d_0 d_1 + d_1^2 and E = d_0 d_1 (d_0 + d_1) = -d_0 d_1 d_2 alone, and since d_k is a root of
x^3 = p x - E, every Y_k is a quadratic in d_k with symmetric coefficients:

    J   = A + i E B,          Y_k = alpha + beta d_k + gamma d_k^2,
    beta  = i bi + E br,      gamma = gr + i E gi,      alpha = (J - 2 p gamma) / 3   (sum_k Y_k = J),

A, B, bi, br, gr, gi real functions of p and w = E^2. Their Taylor coefficients are rational and formed
exactly below; each function is then fitted on the phases max |d_k| <= M by a polynomial
sum_c w^c sum_a c_a p^a with the given number of terms per power of w (w <= 4 p^3 / 27, so few are
needed), the largest error (times |E| for B, br, gi) minimised by Lawson's reweighted least squares in
80-bit arithmetic. Symmetric functions in two variables need about half the operations of the
one-variable recurrences in n.

Four sets: binary32 J in the scaled phases d / (4 pi) (half-phases in turns), binary32 moments, binary64 and binary64
for short phases in radians. The binary64 sine and cosine on [-pi/4, pi/4] (their arguments are reduced by multiples of pi/2) are fitted the same way:
sin x = x + x^3 S(x^2), cos x = 1 - x^2 / 2 + x^4 C(x^2).
Run from this directory (on a machine with an 80-bit long double): python gen_face_poly.py > face_poly.h
"""
from fractions import Fraction
from math import comb, factorial

import numpy as np

LD = np.longdouble
NMAX = 44

# (terms in p for w^0, w^1, ...) of each function, and the phase range
M32, M64, M64S = 3.6, 3.0, 1.5
SHAPE32 = {"A": (6, 3), "B": (5, 2)}                     # the forward's J, phases to M32
SHAPE32M = {"A": (6, 3), "B": (5, 2), "bi": (5, 2), "br": (4, 1), "gr": (5, 2), "gi": (3,)}  # moments, to M64
SHAPE64 = {"A": (11, 8, 4, 1), "B": (9, 6, 3), "bi": (9, 7, 3, 1), "br": (8, 5, 2), "gr": (9, 6, 3), "gi": (8, 4, 1)}
SHAPE64S = {"A": (8, 5, 2), "B": (7, 4, 1), "bi": (7, 4, 1), "br": (6, 3), "gr": (7, 4, 1), "gi": (6, 3)}  # to M64S
ODD = ("B", "br", "gi")  # multiplied by E
ROW64 = []  # every binary64 coefficient, in the order of the "at" offsets


def taylor():
    """{function: {(a, c): coefficient of p^a w^c}} to total degree NMAX in d, exact."""
    out = {k: {} for k in SHAPE64}

    def add(name, a, c, v):
        out[name][(a, c)] = out[name].get((a, c), Fraction(0)) + v

    # h_n(d) = sum over 2a + 3b = n of C(a+b, a) p^a e3^b, e3 = d_0 d_1 d_2 = -E
    h = [{((n - 3 * b) // 2, b): comb((n - 3 * b) // 2 + b, b) for b in range(n // 3 + 1) if (n - 3 * b) % 2 == 0}
         for n in range(NMAX + 1)]
    sign = [1, 1, -1, -1]  # i^n = sign (n even) or i sign (n odd)
    for n in range(NMAX + 1):
        for (a, b), v in h[n].items():
            if n % 2 == 0:
                add("A", a, b // 2, sign[n % 4] * Fraction(v, factorial(n + 2)))
            else:
                add("B", a, (b - 1) // 2, -sign[n % 4] * Fraction(v, factorial(n + 2)))
    # x^j mod (x^3 - p x - e3) = r_j + s_j x + t_j x^2, as {(power of p, power of e3): integer}
    def mul(f, a0, b0):
        return {(a + a0, b + b0): v for (a, b), v in f.items()}

    def plus(f, g):
        s = dict(f)
        for k, v in g.items():
            s[k] = s.get(k, 0) + v
        return s
    r, s, t = [{(0, 0): 1}], [{}], [{}]
    for j in range(NMAX):
        r.append(mul(t[j], 0, 1))
        s.append(plus(r[j], mul(t[j], 1, 0)))
        t.append(dict(s[j]))
    # h_n(d, x) = sum_j h_{n-j}(d) x^j
    for n in range(NMAX + 1):
        for j in range(n + 1):
            for (a, b), v in h[n - j].items():
                for part, even, odd in ((s[j], "br", "bi"), (t[j], "gr", "gi")):
                    for (a2, b2), v2 in part.items():
                        val = sign[n % 4] * Fraction(v * v2, factorial(n + 3))
                        aa, bb = a + a2, b + b2
                        name = odd if n % 2 else even
                        if name in ODD:
                            add(name, aa, (bb - 1) // 2, -val)
                        else:
                            add(name, aa, bb // 2, val)
    return out


def value(T, p, w):
    """Taylor polynomial at (p, w), 80-bit."""
    s = np.zeros_like(p)
    for c in range(max(c for _, c in T) + 1):
        col = [T.get((a, c), Fraction(0)) for a in range(NMAX // 2 + 1)]
        h = np.zeros_like(p)
        for v in reversed(col):
            h = h * p + LD(v.numerator) / LD(v.denominator)
        s = s + h * w ** c
    return s


def grid(M, ns=40, nt=15):
    """Phases (d_0, d_1) with max |d| <= M: Chebyshev points in p times triangle shapes (up to symmetry)."""
    out = []
    for i in range(ns):
        m = LD(M) * np.sqrt((1 - np.cos(LD(np.pi) * (i + 0.5) / ns)) / 2)
        for j in range(nt):
            a = LD(np.pi) / 6 * (1 - np.cos(LD(np.pi) * j / (nt - 1)))
            d = [np.cos(a + k * 2 * LD(np.pi) / 3) for k in range(3)]
            k = m / max(abs(x) for x in d)
            out.append((d[0] * k, d[1] * k))
    out = np.array(out, LD)
    return out[:, 0], out[:, 1]


def least_squares(A, y):
    A, y = A.copy(), y.copy()
    n = A.shape[1]
    for k in range(n):  # Householder
        v = A[k:, k].copy()
        v[0] += np.sqrt((v * v).sum()) * (1 if v[0] >= 0 else -1)
        v /= np.sqrt((v * v).sum())
        A[k:, k:] -= 2 * np.outer(v, v @ A[k:, k:])
        y[k:] -= 2 * v * (v @ y[k:])
    c = np.zeros(n, LD)
    for k in reversed(range(n)):
        c[k] = (y[k] - (A[k, k + 1:] * c[k + 1:]).sum()) / A[k, k]
    return c


def fit(T, M, shape, odd, exact0, rounds=30):
    """{(a, c): coefficient of p^a w^c} and the largest error on the grid (times |E| if odd). exact0: the
    constant term is the function's value at 0 (J's 1/2, whose rounding would scale every small face)."""
    d0, d1 = grid(M)
    p, E = d0 * d0 + d0 * d1 + d1 * d1, d0 * d1 * (d0 + d1)
    w = E * E
    y, unit = value(T, p, w), (abs(E) if odd else np.ones_like(p))
    P, W = p.max(), w.max()
    # Chebyshev basis in p for conditioning, as monomial coefficients for the result
    nmax = max(shape)
    tm = [np.array([1], LD), np.array([-1, 2 / P], LD)]
    tv = [np.ones_like(p), 2 * p / P - 1]
    for k in range(2, nmax):
        a = np.zeros(k + 1, LD)
        a[1:] += 4 / P * tm[-1]
        a[:k] -= 2 * tm[-1]
        a[:k - 1] -= tm[-2]
        tm.append(a)
        tv.append(2 * tv[1] * tv[-1] - tv[-2])
    mon = [(a, c) for c, na in enumerate(shape) for a in range(na)]
    basis = [tv[a] * (w / W) ** c for a, c in mon]
    c0 = LD(T[(0, 0)].numerator) / LD(T[(0, 0)].denominator)
    if exact0:  # the constant term is kept: p T_a(p) instead of T_{a+1}(p) for w^0
        mon = [m for m in mon if m != (shape[0] - 1, 0)]
        basis = [p / P * tv[a] if c == 0 else tv[a] * (w / W) ** c for a, c in mon]
        y = y - c0
    A = np.stack(basis, 1)
    lw, best = np.ones(len(y), LD) / len(y), None
    for _ in range(rounds):
        sw = np.sqrt(lw) * unit
        c = least_squares(A * sw[:, None], y * sw)
        r = abs(A @ c - y) * unit
        if best is None or r.max() < best[0]:
            best = (r.max(), c)
        lw = np.maximum(lw * r / (lw * r).sum(), LD(1e-25))
    res = {}
    for (a, c), v in zip(mon, best[1]):
        for k, x in enumerate(tm[a]):
            k, x = (k + 1, x / P) if exact0 and c == 0 else (k, x)
            res[(k, c)] = res.get((k, c), LD(0)) + v * x / W ** c
    if exact0:
        res[(0, 0)] = c0
    return res, float(best[0])


def table(name, T, M, shape, odd, scale, kind):
    """Lines of one function's coefficient arrays; scale s: the variables are d / s (p / s^2, E / s^3)."""
    c, err = fit(T, M, shape, odd, name == "A")
    out = [f"  // error {err:.1e}" + (" (times |E|)" if odd else "")]
    for k, na in enumerate(shape):
        v = [c[(a, k)] * LD(scale) ** (2 * a + 6 * k + (3 if odd else 0)) for a in range(na)]
        if kind == "float":
            txt = ", ".join(f"{float(np.float32(x))!r}f" for x in v)
        else:
            txt = ", ".join(repr(float(x)) for x in v)
        at = ""
        if kind == "double":
            at = f" static constexpr int at = {len(ROW64)};"
            ROW64.extend(repr(float(x)) for x in v)
        out.append(f"  struct {name}{k} {{ static constexpr {kind} c[{na}] = {{{txt}}};{at} }};")
    return out


def sincos_fit(first, terms, rounds=40):
    """Coefficients of g(z), z = x^2, with first = 3: sin x = x + x^3 g, first = 4: cos x = 1 - x^2/2 + x^4 g,
    on |x| <= pi/4 (error of the sine or cosine minimised)."""
    n = 400
    z = (LD(np.pi) / 4 * LD(1.0001)) ** 2 * (1 - np.cos(LD(np.pi) * (np.arange(n, dtype=LD) + LD(0.5)) / n)) / 2
    y = np.zeros(n, LD)
    for k in reversed(range(14)):
        y = y * z + LD((-1) ** (k + (1 if first == 3 else 0))) / LD(factorial(first + 2 * k))
    unit = z ** (LD(first) / 2)
    A = np.stack([(z / z.max()) ** a for a in range(terms)], 1)
    lw, best = np.ones(n, LD) / n, None
    for _ in range(rounds):
        sw = np.sqrt(lw) * unit
        c = least_squares(A * sw[:, None], y * sw)
        r = abs(A @ c - y) * unit
        if best is None or r.max() < best[0]:
            best = (r.max(), c)
        lw = np.maximum(lw * r / (lw * r).sum(), LD(1e-25))
    return [float(v / z.max() ** a) for a, v in enumerate(best[1])], float(best[0])


def main():
    T = taylor()
    print("// Generated by gen_face_poly.py; do not edit.")
    print("// Fitted polynomials of a triangle's face integral J = A + i E B and of its barycentric moments")
    print("// Y_k = alpha + beta d_k + gamma d_k^2 (beta = i bi + E br, gamma = gr + i E gi, alpha = (J - 2 p gamma) / 3)")
    print("// for centred vertex phases max |d_k| <= M: each function is sum_k w^k sum_a f<k>::c[a] p^a with")
    print("// p = d_0^2 + d_0 d_1 + d_1^2, E = d_0 d_1 (d_0 + d_1), w = E^2. \"error\" is the fit's largest.")
    print("#pragma once\n\nnamespace pft {\n")
    print("// sin x = x + x^3 S(x^2), cos x = 1 - x^2 / 2 + x^4 C(x^2) on [-pi/4, pi/4], binary64.")
    print("struct SinCos64 {")
    for name, first in (("S", 3), ("C", 4)):
        c, err = sincos_fit(first, 6)
        print(f"  // error {err:.1e}")
        print(f"  struct {name} {{ static constexpr double c[{len(c)}] = {{{', '.join(repr(v) for v in c)}}};"
              f" static constexpr int at = {len(ROW64)}; }};")
        ROW64.extend(repr(v) for v in c)
    print("};\n")
    for st, M, shapes, scale, kind, what in (
            ("FaceFit32", M32, SHAPE32, LD(4) * LD("3.14159265358979323846264338"), "float",
             "binary32; the variables are phases / (4 pi): p, E, w of d / (4 pi)"),
            ("FaceFit32M", M64, SHAPE32M, 1, "float", "binary32 moments; phases in radians"),
            ("FaceFit64", M64, SHAPE64, 1, "double", "binary64; phases in radians"),
            ("FaceFit64S", M64S, SHAPE64S, 1, "double", "binary64, short phases in radians")):
        print(f"// {what}; M in radians.")
        print(f"struct {st} {{")
        print(f"  static constexpr double M = {M!r};")
        for name in shapes:
            # beta and gamma multiply d_k and d_k^2, which carry their own scale
            for line in table(name, T[name], M, shapes[name], name in ODD, scale, kind):
                print(line)
        print("};\n")
    print("// Every binary64 coefficient above in one row; a function's start at its \"at\".")
    print("#define PFT_FIT64_ROW \\")
    rows = [", ".join(ROW64[i:i + 5]) for i in range(0, len(ROW64), 5)]
    print(", \\\n".join("  " + r for r in rows))
    print("\n}  // namespace pft")


if __name__ == "__main__":
    main()
