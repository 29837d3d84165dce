"""Layouts that a batch's FP64 kernel and its last group take by the number of cells: the results do not
depend on them, and a batch takes no longer than one with more cells."""
import statistics

import numpy as np
import pytest
import torch

from paper_1211_0540_amd import bz
from paper_1211_0540_amd import workloads as W

pytestmark = pytest.mark.gpu
_WCACHE = {}


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch.device("cuda:0")


def _batch(N, L, cells, mode, dev):
    c = bz.Collision([(N, L, 1.0)], [0] * len(cells), mode, weights_cache=_WCACHE)
    return c, torch.from_numpy(c.pack(cells)).to(dev)


def _time(fn):
    """Median time of a call in ms, over ten groups of calls."""
    for _ in range(3):
        fn()
    times = []
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            fn()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) / 5)
    return statistics.median(times)


# a narrow group alone, whole groups with a narrow one, whole groups alone: the same cells, bitwise
@pytest.mark.parametrize("N,L", [(16, 6.0), (20, 6.0)])
def test_fp64_forms_agree_bitwise(dev, N, L):
    base = list(W.random_smooth_cells(20, N, L, seed=600 + N, umax=0.5))
    cells = [base[i % 20] * (1.0 + i / 256) for i in range(128)]
    out = {}
    for n in (20, 64, 84, 128):
        c, f = _batch(N, L, cells[:n], "batched_f64", dev)
        out[n] = c.collide(f).cpu().numpy()
        c.close()
    assert np.all(np.isfinite(out[128]))
    for n in (20, 64, 84):
        assert np.array_equal(out[n], out[128][:n * N ** 3])


# the widest narrow group against a whole group of the same mesh: half the cells in at most its
# time (equal where both run the whole layout; 10% for the clock)
@pytest.mark.parametrize("N,L", [(24, 7.0), (28, 7.0), (32, 8.0)])
def test_fp64_half_group_takes_no_longer_than_a_whole_one(dev, N, L):
    base = W.random_smooth_cells(1, N, L, seed=700 + N, umax=0.5)[0]
    ms = {}
    for n in (32, 64):
        c, f = _batch(N, L, [base] * n, "batched_f64", dev)
        q = torch.empty_like(f)
        ms[n] = _time(lambda: c.collide(f, q))
        c.close()
    assert ms[32] <= 1.1 * ms[64], ms
