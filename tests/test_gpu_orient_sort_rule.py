"""Which orientation averages sort their Q list: those of fewer than 256 directions, and the binary64 ones of 1e8 pairs or
more, whose wavefronts of short and long phases cost more than the sort (224 faces x 819 200 Q: 0.85 ms sorted, 0.93 to
1.01 as listed)."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,nqa,ndir,sort", [("fp64", 400, 2048, True), ("fp64", 100, 2048, False),
                                                ("fp32c", 400, 2048, False), ("fp32c", 100, 255, True),
                                                ("fp64", 100, 255, True), ("fp64", 20, 255, False)])
def test_sort_rule(gpu, mode, nqa, ndir, sort):
    v, t = mg.ellipsoid_uv([46.0, 31.0, 23.0], 8)  # 224 faces
    rng = np.random.default_rng(1)
    d = rng.normal(size=(ndir, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    args = dev(v), dev(t, torch.int32), dev(np.linspace(0.0, 0.5, nqa)), dev(d), dev(np.full(ndir, 1.0 / ndir))
    step(f"{nqa} magnitudes x {ndir} directions {mode}")
    pft.orientation_average(*args, mode=mode)
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        pft.orientation_average(*args, mode=mode)
        torch.cuda.synchronize()
    names = [e.name for e in p.events()]
    assert any("fwd3d_" in n for n in names), names
    assert any("sort_scatter_kernel" in n for n in names) == sort
