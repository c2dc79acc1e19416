"""The Q order of long lists, whose tiles are sorted in LDS before they are written: sizes about the line and about its
tiles, many equal keys, infinities, and batches of several passes, against a stable sort on the host; and its cost, which must
not grow faster than the list (4e6 random Q took 2.9 times 1e6 when each item was written by itself)."""
import numpy as np
import pytest
import torch

import meshgen as mg
import paper_2104_08309_amd as pft
from gpu_util import dev, host, nrel, step
from test_gpu_qsort import _codes

pytestmark = pytest.mark.gpu
LINE = 3 << 19


@pytest.mark.parametrize("nq", [LINE - 1, LINE, LINE + 1, LINE + 4095, LINE + 4096, LINE + 4097, 2_500_001])
def test_order_is_the_stable_sort(gpu, nq):
    rng = np.random.default_rng(nq)
    for name, q in (("random", rng.random((nq, 3)) - 0.5), ("few points", rng.normal(size=(5, 3))[rng.integers(0, 5, nq)])):
        step(f"q order {name} {nq}")
        got = pft.q_order(dev(q)).cpu().numpy().astype(np.int64)
        assert np.array_equal(got, np.argsort(_codes(q), kind="stable")), name


def test_long_batch(gpu):
    """Five boxes of unequal lists (3 bits of mesh, three passes), one list of most of the Q."""
    v, t = mg.box(1.0, 1.3, 0.7)
    n = [1000, 1_600_000, 3, 90_000, 65]
    rng = np.random.default_rng(1)
    q = np.concatenate([mg.q_random_ball(k, 3.0 * (i + 1), rng) for i, k in enumerate(n)])
    off = np.concatenate([[0], np.cumsum(n)])
    step("batch of long lists")
    F = host(pft.batch_forward(dev(np.tile(v, (5, 1))), dev(np.tile(t, (5, 1)), torch.int32), dev(q),
                               np.arange(6) * len(v), np.arange(6) * len(t), off, mode="fp64"))
    L = np.array([1.0, 1.3, 0.7])
    h = 0.5 * q * L
    want = (L * np.sinc(h / np.pi) * np.exp(1j * h)).prod(axis=1)
    for i in range(5):
        s = slice(off[i], off[i + 1])
        assert nrel(F[s], want[s]) < 1e-12


def test_cost_per_q(gpu):
    torch.manual_seed(1)
    us = []
    for nq in (1_000_000, 4_000_000):
        q = torch.rand(nq, 3, device="cuda") - 0.5
        best = np.inf
        for k in range(15):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(4):
                pft.q_order(q)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, 250.0 * e[0].elapsed_time(e[1]))
        step(f"order of {nq} Q: {best:.1f} us")
        us.append(best)
    assert us[1] < 2.2 * us[0], us
