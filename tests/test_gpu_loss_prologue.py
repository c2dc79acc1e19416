"""The FP32C intensity loss with a face order makes two sets of records of one mesh: its centre and radius are formed
once, on both sides of the size from which they take several blocks, and the values are those of the list order."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import TOL_FP32C, dev, host, nrel, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level", [2, 4, 5])  # 162, 2 562 and 10 242 vertices: one launch, one block, several blocks
def test_centre_once(gpu, level):
    v, t = mg.icosphere(level, 2.0)
    rng = np.random.default_rng(level)
    q = dev(mg.q_random_ball(500, 3.0, rng))
    V, T, target = dev(v), dev(t, torch.int32), dev(rng.random(500))
    order = tuple(dev(x) for x in pft.strip_order(t, len(v)))
    run = lambda o: pft.intensity_loss_3d(V, T, q, target, mode="fp32c", order=o)  # noqa: E731
    step(f"ordered loss, {len(t)} faces")
    loss, grad = run(order)
    step("in the list order")
    loss0, grad0 = run(None)
    assert abs(float(loss) - float(loss0)) < 10 * TOL_FP32C * float(loss0)
    assert nrel(host(grad), host(grad0)) < 10 * TOL_FP32C
    step("under the profiler")
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        run(order)
        torch.cuda.synchronize()
    names = [e.name for e in p.events()]
    assert any("fwd3d_fp32c" in n for n in names), names
    assert sum(any(k in n for k in ("mesh_info_kernel", "centre_radius_kernel", "mesh_records_small_kernel"))
               for n in names) == 1, names
