"""Narrow last groups of the one-launch convolution (at most 32 cells, W = 4, 8, 16 or 32 lanes of
cells and 64 / W steps at once) against the same cells in 64-cell groups: the per-mesh launches
with the same accumulation variant use the wide layout for every group.  The partial sums of a
narrow item are added in step order, so the results are bitwise equal."""
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


# widths 4, 8, 16, 32 at their first and last cell counts, alone and after a full group, on every mesh
@pytest.mark.parametrize("N,L,n,schedule", [
    (8, 4.0, 1, "symmetric"), (8, 4.0, 96, "full"), (12, 5.0, 5, "symmetric"), (12, 5.0, 68, "full"),
    (16, 6.0, 4, "symmetric"), (16, 6.0, 9, "full"), (20, 6.0, 8, "symmetric"), (20, 6.0, 81, "symmetric"),
    (24, 7.0, 16, "full"), (24, 7.0, 72, "symmetric"), (28, 7.0, 17, "symmetric"), (28, 7.0, 1, "full"),
    (32, 8.0, 32, "symmetric"), (32, 8.0, 3, "symmetric"), (32, 8.0, 33, "symmetric")])
def test_narrow_groups_are_bitwise_the_wide_ones(dev, N, L, n, schedule):
    cells = list(W.random_smooth_cells(n, N, L, seed=300 + N, umax=0.5))
    out = []
    for per_mesh in (False, True):
        c = bz.Collision([(N, L, 1.0)], [0] * n, "batched_f32", weights_cache=_WCACHE, schedule=schedule,
                         per_mesh=per_mesh)
        assert bz.bz_batch_one_launch(c.batch) != per_mesh
        c.set_variant(12)
        f = torch.from_numpy(c.pack(cells)).to(dev)
        out.append(c.collide(f).cpu().numpy())
        c.close()
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[1])


# FP64: a narrow item adds the steps' partials in step order as well (bitwise)
@pytest.mark.parametrize("N,L,n", [(8, 4.0, 2), (12, 5.0, 67), (16, 6.0, 32), (20, 6.0, 6), (24, 7.0, 17), (28, 7.0, 4),
                                   (32, 8.0, 9)])
def test_narrow_groups_fp64_are_bitwise_the_wide_ones(dev, N, L, n):
    cells = list(W.random_smooth_cells(n, N, L, seed=400 + N, umax=0.5))
    wide = cells + [cells[0]] * (33 + n // 64 * 64 - n if n % 64 < 33 else 0)   # a last group of 33 cells is wide
    out = []
    for fs in (cells, wide):
        c = bz.Collision([(N, L, 1.0)], [0] * len(fs), "batched_f64", weights_cache=_WCACHE, fine_split=True)
        f = torch.from_numpy(c.pack(fs)).to(dev)
        out.append(c.collide(f).cpu().numpy()[:n * N ** 3])
        c.close()
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[1])


# one queue and a queue per XCD (from three groups and 13 MB of fhat rows on): the smallest batch of N = 16
# on the upper side of the line and one below it, a narrow last group, a batch of three groups
@pytest.mark.parametrize("N,L,n", [(16, 6.0, 400), (16, 6.0, 330), (24, 7.0, 160), (28, 7.0, 129)])
def test_queues_are_bitwise_the_per_mesh_launch(dev, N, L, n):
    base = W.random_smooth_cells(20, N, L, seed=500 + N, umax=0.5)
    cells = [base[i % 20] * (1.0 + i / 1024) for i in range(n)]
    out = []
    for per_mesh in (False, True):
        c = bz.Collision([(N, L, 1.0)], [0] * n, "batched_f32", weights_cache=_WCACHE, per_mesh=per_mesh)
        assert bz.bz_batch_one_launch(c.batch) != per_mesh
        c.set_variant(12)
        f = torch.from_numpy(c.pack(cells)).to(dev)
        for _ in range(2):
            out.append(c.collide(f).cpu().numpy())
        c.close()
    assert np.all(np.isfinite(out[0]))
    for o in out[1:]:
        assert np.array_equal(out[0], o)
