"""Steps of pass A of the conjugate-symmetric schedule whose rows lie on a zeroed plane of its fhat copy
(m2 = 0 or j2 = k2 + N/2 - m2 = 0) add nothing and are left out: with weights that are not
numbers in their place, which no other pass reads, the results are bitwise the same."""
import numpy as np
import pytest
import torch

from paper_1211_0540_amd import bz
from paper_1211_0540_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch.device("cuda:0")


def _unread_steps(N):
    """Indices, in the batched weight stream, of the steps that pass A leaves out."""
    h, at, out = N // 2, 0, []
    lo, hi = (lambda k: max(0, k - h + 1)), (lambda k: min(N - 1, k + h))
    for k1 in range(N):
        for k2 in range(N):
            derived = k1 >= 1 and k2 >= 1 and (k1 > h or (k1 == h and k2 > h))
            for m1 in range(lo(k1), min((k1 + h) // 2, hi(k1)) + 1):
                for m2 in range(lo(k2), (hi(k2) if 2 * m1 < k1 + h else min((k2 + h) // 2, hi(k2))) + 1):
                    if not derived and m1 > 0 and (m2 == 0 or k2 + h - m2 == 0):
                        out.append(at)
                    at += 1
    return np.array(out)


@pytest.mark.parametrize("mode,N,L,n", [("batched_f32", 16, 6.0, 64), ("batched_f32", 24, 7.0, 40), ("batched_f32", 28, 7.5, 64),
                                        ("batched_f32", 32, 8.0, 40), ("batched_f64", 20, 6.0, 64),
                                        ("batched_f64", 24, 7.0, 64), ("batched_f64", 32, 8.0, 40),
                                        ("batched_f64", 20, 6.0, 16), ("batched_f64", 24, 7.0, 72),
                                        ("batched_f64", 28, 7.5, 3)])
def test_steps_on_a_zeroed_plane_are_left_out(dev, mode, N, L, n):
    base = W.random_smooth_cells(4, N, L, seed=900 + N, umax=0.5)
    c = bz.Collision([(N, L, 1.0)], [0] * n, mode)
    f = torch.from_numpy(c.pack([base[i % 4] * (1.0 + i / 256) for i in range(n)])).to(dev)
    want = c.collide(f).cpu().numpy()
    slots = 3 * N * N // 4
    w = c.weights[0].view(torch.float32 if mode == "batched_f32" else torch.float64)
    idx = torch.from_numpy(_unread_steps(N)).to(dev)[:, None] * slots + torch.arange(slots, device=dev)[None, :]
    assert torch.all(torch.isfinite(w[idx.reshape(-1)]))
    w[idx.reshape(-1)] = float("nan")
    got = c.collide(f).cpu().numpy()
    c.close()
    assert np.all(np.isfinite(want))
    assert np.array_equal(got, want)
