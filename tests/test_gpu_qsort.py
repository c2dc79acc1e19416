"""The Q order's radix sort against a stable sort of the same Morton codes on the host: sizes around its tiles and the
smallest sorted list, many equal keys, NaN coordinates."""
import numpy as np
import pytest
import torch

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, step

pytestmark = pytest.mark.gpu


def _codes(q):
    lo, hi = np.nanmin(q, axis=0), np.nanmax(q, axis=0)
    ext = hi - lo
    code = np.zeros(len(q), dtype=np.int64)
    for k in range(3):
        u = (q[:, k] - lo[k]) / ext[k] * 32.0 if ext[k] > 0 else np.zeros(len(q))
        u = np.clip(np.where(np.isnan(u), 0.0, u), 0.0, 31.0).astype(np.int64)
        for b in range(5):
            code |= ((u >> b) & 1) << (3 * b + k)
    return code


@pytest.mark.parametrize("nq", [8192, 8193, 12287, 12288, 40961, 300001])
def test_order_is_the_stable_sort(gpu, nq):
    rng = np.random.default_rng(nq)
    for name, q in (("ball", mg.q_random_ball(nq, 0.5, rng)),
                    ("plane", np.c_[rng.normal(size=(nq, 2)), np.zeros(nq)]),
                    ("few points", rng.normal(size=(5, 3))[rng.integers(0, 5, nq)]),
                    ("nan", np.where(rng.random((nq, 3)) < 0.01, np.nan, rng.normal(size=(nq, 3))))):
        step(f"q order {name} {nq}")
        got = pft.q_order(dev(q)).cpu().numpy().astype(np.int64)
        assert np.array_equal(got, np.argsort(_codes(q), kind="stable")), name
