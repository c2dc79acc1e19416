"""The Q order of a batch: each list by its own cells. Lists of unequal range, outlying, NaN and infinite Q and lists of a
few Q give the values of the meshes alone; an outlying Q in each list does not undo the order of the others (the
binary64 adjoint of lists about its phase limit costs half as much again in the list order)."""
import numpy as np
import pytest
import torch

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, host, nrel, step

pytestmark = pytest.mark.gpu


def _off(x):
    return np.concatenate([[0], np.cumsum([len(y) for y in x])]).astype(np.int64)


def _hull(rng, k, r):
    p = rng.normal(size=(k, 3))
    return mg.convex_hull_mesh(p * (r / np.linalg.norm(p, axis=1))[:, None])


def _pack(meshes, qs):
    vs, ts = [v for v, _ in meshes], [t for _, t in meshes]
    return (dev(np.concatenate(vs)), dev(np.concatenate(ts), torch.int32), dev(np.concatenate(qs)), _off(vs), _off(ts),
            _off(qs))


def test_values(gpu):
    """(In binary64: the order is the same in both forms, and there it is the only difference that could show.)"""
    mode, tol = "fp64", 1e-12
    rng = np.random.default_rng(1)
    meshes, qs = [], []
    for n in (3, 64, 65, 700, 1, 5000, 3001, 0, 1023, 1025, 900):
        r = float(np.exp(rng.uniform(np.log(2.0), np.log(60.0))))
        meshes.append(_hull(rng, int(rng.integers(8, 60)), r))
        q = mg.q_random_ball(n, 12.0 / r, rng)
        if n > 100:
            q[rng.integers(0, n, 3)] *= 4.0
        qs.append(q)
    qs[3][:, 1] = 0.0                                   # a slice
    qs[5][:] = qs[5][rng.integers(0, 4, 5000)]          # few different points
    bad = [(qs[6], 7, np.nan), (qs[6], 11, np.inf), (qs[9], 0, -np.inf), (qs[2], 64, np.inf)]
    for q, i, x in bad:
        q[i, 2] = x
    args = _pack(meshes, qs)
    step(f"batch of unequal lists, forward {mode}")
    F = host(pft.batch_forward(*args, mode=mode))
    finite = np.isfinite(np.concatenate(qs)).all(axis=1)
    assert np.array_equal(np.isnan(F), ~finite)
    c = rng.normal(size=len(F)) + 1j * rng.normal(size=len(F))
    c[~finite] = 0.0
    clean = [np.where(np.isfinite(q), q, 0.1) for q in qs]
    args = _pack(meshes, clean)
    step("the same with finite Q, adjoint")
    G = host(pft.batch_backward(*args, dev(c), mode=mode))
    for i, (v, t) in enumerate(meshes):
        s = slice(args[5][i], args[5][i + 1])
        if s.stop == s.start:
            assert not G[args[3][i]:args[3][i + 1]].any()
            continue
        step(f"mesh {i} alone: {len(t)} faces, {s.stop - s.start} Q")
        one = host(pft.forward_3d(dev(v), dev(t, torch.int32), dev(qs[i]), mode=mode))
        ok = finite[s]
        assert nrel(F[s][ok], one[ok]) < tol
        g = host(pft.backward_3d(dev(v), dev(t, torch.int32), dev(clean[i]), dev(c[s]), mode=mode))
        assert nrel(G[args[3][i]:args[3][i + 1]], g) < 10 * tol


def test_lists_of_one(gpu):
    """More meshes than leave five bits an axis to the cells: an infinite Q must not carry into the next mesh's key."""
    n = (1 << 17) + 5
    v, t = mg.box(1.0, 1.3, 0.7)
    rng = np.random.default_rng(2)
    q = mg.q_random_ball(n, 4.0, rng)
    scale = 0.5 + rng.random(n)
    q[::1000] = np.inf
    V = (v[None] * scale[:, None, None]).reshape(-1, 3)
    T = np.tile(t, (n, 1))
    step(f"{n} boxes of one Q each")
    F = host(pft.batch_forward(dev(V), dev(T, torch.int32), dev(q), np.arange(n + 1) * len(v),
                               np.arange(n + 1) * len(t), np.arange(n + 1), mode="fp64"))
    ok = np.isfinite(q[:, 0])
    assert np.isnan(F[~ok]).all()
    # box of edges L: prod L sinc(Q L / 2) exp(i Q L / 2)
    L = np.array([1.0, 1.3, 0.7])[None] * scale[:, None]
    h = 0.5 * q[ok] * L[ok]
    want = (L[ok] * np.sinc(h / np.pi) * np.exp(1j * h)).prod(axis=1)
    assert nrel(F[ok], want) < 1e-12


def test_outlying_q_keeps_the_order(gpu):
    """Lists of short and long Q by turns, which cost little only where the order parts them, without and with two Q at
    30 times the range: the same time, but for their own wavefronts. (1.38 times with cells in the box of all Q.)"""
    rng = np.random.default_rng(3)
    meshes = [_hull(rng, 60, 40.0) for _ in range(12)]
    qs = [mg.q_random_ball(24000, 0.5, rng) for _ in meshes]
    for q in qs:
        q *= (np.where(np.arange(24000) % 2, 0.5, 0.025) / np.linalg.norm(q, axis=1))[:, None]
    c = dev(rng.normal(size=24000 * 12) + 0j)
    ms = []
    for scale in (1.0, 30.0):
        for q in qs:
            q[17] = np.array([0.25, 0.1, 0.15]) * scale
            q[19] = -q[17]
        args = _pack(meshes, qs)
        best = np.inf
        for k in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            pft.batch_backward(*args, c, mode="fp64")
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        step(f"adjoint, two Q a list at {scale:g} times the range: {best:.3f} ms")
        ms.append(best)
    assert ms[1] < 1.15 * ms[0], ms


def test_outlying_q_of_one_list(gpu):
    """The same for one list through the order itself: the wavefronts of its short Q stay short (in equal cells of the box
    of all Q two in three held both kinds), and those of a list without outlying Q."""
    rng = np.random.default_rng(4)
    n = 24000
    q = mg.q_random_ball(n, 0.5, rng)
    q *= (np.where(np.arange(n) % 2, 0.5, 0.025) / np.linalg.norm(q, axis=1))[:, None]
    for outlying in (0, 2, 40):
        x = q.copy()
        x[:outlying] *= 30.0
        step(f"order of a list with {outlying} outlying Q")
        order = pft.q_order(dev(x)).cpu().numpy().astype(np.int64)
        assert np.array_equal(np.sort(order), np.arange(n))
        long = (order % 2 == 1)[: n // 64 * 64].reshape(-1, 64)
        mixed = np.mean(long.any(axis=1) & ~long.all(axis=1))
        print(f"mixed wavefronts: {mixed:.3f}")
        assert mixed < 0.1
