"""Lists of small Q alone in binary64: their wavefronts sum the tetrahedron fans and no surface terms. Values against the
oracle about the sizes of a wavefront, a Q tile and the lane-per-face limit, by mesh, region and batch; and the time of the
kernels against that of a list of Q just beyond the fans (with both sums it was half as long again to twice as long)."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP64, dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 9, 64, 65, 73, 128, 137, 300])
@pytest.mark.parametrize("n_lat", [3, 11])  # 24 and 440 faces
def test_values(gpu, n_lat, n):
    v, t = mg.ellipsoid_uv([1.3, 1.0, 0.8], n_lat, centre=(0.2, -0.1, 0.3))
    rng = np.random.default_rng(n_lat + n)
    q = mg.q_random_ball(n, 0.004, rng)
    A, B = dev(v), dev(t, torch.int32)
    F, dF = O.ft3d(v, t, q), O.ft3d_dq(v, t, q)
    step(f"{len(t)} faces, {n} small Q")
    got = host(pft.forward_3d(A, B, dev(q), mode="fp64"))
    assert nrel(got, F) < TOL_FP64
    q5 = np.r_[q, mg.q_random_ball(200, 5.0, rng)]
    mixed = host(pft.forward_3d(A, B, dev(q5), mode="fp64"))[:n]
    assert nrel(mixed, got) < 1e-15 * len(t) ** 0.5  # the splits of the sum alone may differ
    v2, t2 = np.r_[v, v + [9.0, 0.0, 0.0]], np.r_[t, t + len(v)]
    Fr, dFr = F + O.ft3d(v + [9.0, 0.0, 0.0], t, q), dF + O.ft3d_dq(v + [9.0, 0.0, 0.0], t, q)
    c = rng.normal(size=n) + 1j * rng.normal(size=n)
    step("two regions")
    args = dev(v2), dev(t2, torch.int32), [0, len(t), 2 * len(t)], dev(np.ones(2)), dev(q)
    assert nrel(host(pft.forward_3d_regions(*args, mode="fp64")), Fr) < TOL_FP64
    gq = pft.backward_3d_regions(*args, dev(c), mode="fp64", need_verts=False, need_rho=False)[2]
    assert nrel(host(gq), np.real(np.conj(c)[:, None] * dFr)) < 1e-10
    step("batch")
    vo, to, qo = [0, len(v), 2 * len(v)], [0, len(t), 2 * len(t)], [0, n, n + len(q5)]
    bt = host(pft.batch_forward(dev(np.r_[v, v]), dev(np.r_[t, t], torch.int32), dev(np.r_[q, q5]), vo, to, qo,
                                mode="fp64"))
    assert nrel(bt, np.r_[F, O.ft3d(v, t, q5)]) < TOL_FP64


def _kernel_us(run, kernel):
    run()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        for _ in range(5):
            run()
        torch.cuda.synchronize()
    return min(e.device_time for e in p.events() if kernel in e.name)


@pytest.mark.parametrize("kernel", ["fwd3d_fp64_kernel", "dq3d_fp64_kernel", "batch_fwd_fp64_kernel"])
def test_time(gpu, kernel):
    v, t = mg.icosphere(4, 50.0)
    A, B = dev(v), dev(t, torch.int32)
    rng = np.random.default_rng(3)
    small = mg.q_random_ball(30000, 1e-5, rng)
    beyond = small * (0.01 / np.linalg.norm(small, axis=1, keepdims=True))
    one, c = dev(np.ones(1)), dev(np.ones(30000, complex))
    us = []
    for q in (dev(small), dev(beyond)):
        run = {"fwd3d_fp64_kernel": lambda: pft.forward_3d(A, B, q, mode="fp64"),  # noqa: B023
               "dq3d_fp64_kernel": lambda: pft.backward_3d_regions(A, B, [0, len(t)], one, q, c, mode="fp64",  # noqa: B023
                                                                   need_verts=False, need_rho=False),
               "batch_fwd_fp64_kernel": lambda: pft.batch_forward(A, B, q, [0, len(v)], [0, len(t)], [0, len(q)],  # noqa: B023
                                                                  mode="fp64")}[kernel]
        step(f"{kernel} of 30 000 Q")
        us.append(_kernel_us(run, kernel))
    print(us)
    assert us[0] < 1.3 * us[1], us
