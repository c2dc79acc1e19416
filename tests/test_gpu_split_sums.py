"""The sums over the adjoint's Q splits, added eight loads at a time: lists of split counts about multiples of eight, for
meshes below and above the size of the one-launch gather and for batches, against the oracle; and the time of the gather
of many splits against the adjoint's own kernel (with one load at a time it took four times as long as it)."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import oracle as O
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, dev, host, maxrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [255, 1793, 2048, 2304, 4096, 4352, 12289])  # 1, 8, 9, 16, ... passes of 256 Q
@pytest.mark.parametrize("mode,tol", [("fp64", 1e-10), ("fp32c", TOL_FP32C)])
def test_values(gpu, nq, mode, tol):
    rng = np.random.default_rng(nq)
    q = mg.q_random_ball(nq, 3.0, rng)
    c = rng.normal(size=nq) + 1j * rng.normal(size=nq)
    v, t = mg.box(1.0, 1.4, 0.8)
    want = O.grad3d(v, t, q, c)
    step(f"box, {nq} Q, {mode}")
    assert maxrel(host(pft.backward_3d(dev(v), dev(t, torch.int32), dev(q), dev(c), mode=mode)), want) < tol
    step("the same box, then 2 040 empty faces: beyond the one-launch gather")
    t2 = np.r_[t, np.zeros((2040, 3), t.dtype)]
    assert maxrel(host(pft.backward_3d(dev(v), dev(t2, torch.int32), dev(q), dev(c), mode=mode)), want) < tol
    step("batch")
    n = nq // 3
    got = host(pft.batch_backward(dev(np.r_[v, v]), dev(np.r_[t, t], torch.int32), dev(q), [0, 8, 16], [0, 12, 24],
                                  [0, n, nq], dev(c), mode=mode))
    assert maxrel(got, np.r_[O.grad3d(v, t, q[:n], c[:n]), O.grad3d(v, t, q[n:], c[n:])]) < tol


def test_time(gpu):
    v, t = mg.box(40.0, 55.0, 31.0)
    q = dev(mg.q_random_ball(6_000_000, 0.5, np.random.default_rng(5)), torch.float32)
    c = torch.ones(6_000_000, dtype=torch.complex64, device=gpu)
    step("12 faces x 6e6 Q, backward")
    run = lambda: pft.backward_3d(dev(v), dev(t, torch.int32), q, c, mode="fp32c")  # noqa: E731
    run()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        for _ in range(3):
            run()
        torch.cuda.synchronize()
    us = {k: min(e.device_time for e in p.events() if k in e.name) for k in ("gather_small_kernel", "bwd3d_fp32c_kernel")}
    print(us)
    assert us["gather_small_kernel"] < 2.0 * us["bwd3d_fp32c_kernel"], us
