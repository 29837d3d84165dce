"""Layouts and launch shapes that go by the number of cells or rows: the results do not depend on them, and a
call takes no longer than one with more work."""
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


# many cells of a small mesh against the same bytes in cells of a larger one (a cell is one block: up to three times)
@pytest.mark.parametrize("N,n", [(8, 4000), (12, 1188)])
def test_moments_of_many_small_cells(dev, N, n):
    ms = {}
    for mesh, cells in ((N, n), (24, n * N ** 3 // 24 ** 3)):
        g = bz.bz_grid_init(mesh, 6.0, 1.0)
        b = bz.bz_batch_create(np.zeros(cells, np.int32), [g], bz.BZ_MODE_PLAIN_F64)
        f = torch.rand(cells * mesh ** 3, dtype=torch.float64, device=dev)
        mom = torch.empty(5 * cells, dtype=torch.float64, device=dev)
        ms[mesh] = _time(lambda: bz.bz_cell_moments(b, f, mom))
        bz.bz_batch_free(b)
        bz.bz_grid_free(g)
    assert ms[N] <= 3.0 * ms[24], ms


# one launch for all cells, a launch for each kind of mesh, and the meshes alone.  Sums of N^3 positive terms in
# another order differ by at most N^3 2^-53 relative; the velocities are differences of such sums over v up to L.
@pytest.mark.parametrize("spec", [((8, 3), (20, 2), (32, 2)), ((8, 600), (12, 5), (20, 40), (28, 3)), ((20, 7),), ((16, 5),)])
def test_moments_by_kind_of_mesh(dev, spec):
    Ls = {8: 4.0, 12: 5.0, 16: 6.0, 20: 6.0, 28: 7.5, 32: 8.0}
    grids = [bz.bz_grid_init(N, Ls[N], 1.0) for N, _ in spec]
    mesh_of = np.repeat(np.arange(len(spec)), [n for _, n in spec])
    rng = np.random.default_rng(5)
    rng.shuffle(mesh_of)
    cells = [rng.uniform(0.1, 1.0, (spec[m][0],) * 3) for m in mesh_of]
    b = bz.bz_batch_create(mesh_of.astype(np.int32), grids, bz.BZ_MODE_PLAIN_F64)
    f = torch.from_numpy(np.concatenate([c.ravel() for c in cells])).to(dev)
    mom = torch.full((5 * len(cells),), float("nan"), dtype=torch.float64, device=dev)
    bz.bz_cell_moments(b, f, mom)
    got = mom.cpu().numpy().reshape(-1, 5)
    for c, m, o in zip(cells, mesh_of, got):
        N, L = spec[m][0], Ls[spec[m][0]]
        dv, tol = 2 * L / N, 4 * N ** 3 * 2.0 ** -53
        v = dv * (np.arange(N) - N // 2)
        rho = c.sum()
        u = [np.tensordot(c, v, axes=([d], [0])).sum() / rho for d in range(3)]
        w2 = sum((v - u[d]).reshape([-1 if e == d else 1 for e in range(3)]) ** 2 for d in range(3))
        assert abs(o[0] - rho * dv ** 3) <= tol * rho * dv ** 3
        assert np.max(np.abs(o[1:4] - u)) <= tol * L
        assert abs(o[4] - (w2 * c).sum() / (3 * rho)) <= tol * 3 * L * L
    bz.bz_batch_free(b)
    for g in grids:
        bz.bz_grid_free(g)


# a hidden layer of 256 against one of 512 (its last product alone is half as long; 10% for the clock and the host)
@pytest.mark.parametrize("N", [16, 24])
def test_backward_of_a_narrow_layer_takes_no_longer(dev, N):
    rows, M, ms = 96, N ** 3, {}
    for hidden in (256, 512):
        net = bz.bz_mlp_create(M, hidden, M)
        params = torch.zeros(bz.bz_mlp_param_bytes(net), dtype=torch.uint8, device=dev)
        master = np.random.default_rng(3).standard_normal(bz.bz_mlp_param_count(net)) * 0.02
        bz.bz_mlp_set_params(net, params, master.astype(np.float32))
        x = torch.randn(rows, M, device=dev).to(torch.bfloat16).view(torch.int16)
        y = torch.randn(rows, M, device=dev)
        work = torch.zeros(bz.bz_mlp_workspace_bytes(net, rows), dtype=torch.uint8, device=dev)
        grad, loss = torch.zeros(master.size, device=dev), torch.zeros(1, device=dev)
        ms[hidden] = _time(lambda: bz.bz_mlp_backward(net, params, x, y, rows, grad, loss, work))
        bz.bz_mlp_free(net)
    assert ms[256] <= 1.1 * ms[512], ms


# a queue per XCD over several meshes, with narrow last groups of 8, 16 and 32 lanes and whole ones, and on both sides of
# the line in bytes, against the per-mesh launches of the same accumulation variant: bitwise
@pytest.mark.parametrize("spec", [((16, 80), (20, 90), (24, 72), (32, 100)), ((24, 70), (32, 150)), ((16, 392),), ((16, 393),),
                                  ((32, 160),)])
def test_queues_over_meshes_are_bitwise_the_per_mesh_launches(dev, spec):
    Ls = {16: 6.0, 20: 6.0, 24: 7.0, 32: 8.0}
    base = {N: W.random_smooth_cells(8, N, Ls[N], seed=800 + N, umax=0.5) for N, _ in spec}
    mesh_of = np.repeat(np.arange(len(spec)), [n for _, n in spec])
    np.random.default_rng(6).shuffle(mesh_of)
    cells = [base[spec[m][0]][i % 8] * (1.0 + i / 1024) for i, m in enumerate(mesh_of)]
    out = []
    for per_mesh in (False, True):
        c = bz.Collision([(N, Ls[N], 1.0) for N, _ in spec], mesh_of, "batched_f32", weights_cache=_WCACHE,
                         per_mesh=per_mesh)
        assert bz.bz_batch_one_launch(c.batch) != per_mesh
        c.set_variant(12)
        f = torch.from_numpy(c.pack(cells)).to(dev)
        for _ in range(2):
            out.append(c.collide(f).cpu().numpy())
        c.close()
    assert np.all(np.isfinite(out[0]))
    for o in out[1:]:
        assert np.array_equal(out[0], o)


# three groups and a half against four: 3.5 times a group's work at most in the time of 4 (6% for the clock)
def test_a_half_group_does_not_hold_up_the_queues(dev):
    base, ms = W.random_smooth_cells(1, 32, 8.0, seed=732, umax=0.5)[0], {}
    for n in (224, 256):
        c, f = _batch(32, 8.0, [base] * n, "batched_f32", dev)
        q = torch.empty_like(f)
        ms[n] = _time(lambda: c.collide(f, q))
        c.close()
    assert ms[224] <= 1.06 * ms[256], ms
