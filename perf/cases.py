"""The work that users of the library have it do, as a list of timed cases.

A case is a dict of plain values.  `listed` gives the fixed cases, `draw` one more of the same
ranges, `prepare` what a program holds before the call (inputs on the GPU, batch, weights,
workspace), `run` one pass through the public entry points, `work` the bytes and operations a
pass cannot do without, and `exact` the same outputs in 64 bits from plain torch and numpy.

Paths:
  step      one Heun step (bz_step) of a batch of cells, the call a space-homogeneous run makes
  strang    one Strang step (bz_strang_step) of a 1-D problem with a heated wall
  closure   one Heun step with the gated learned closure (bz_closure_step)
  collide   one evaluation and its projection (bz_collide_batch, bz_project) in FP64, where Q
            itself is wanted as a reference
  train     forward, gradients and Adam of the closure's network (bz_mlp_backward, bz_mlp_adam)
  serve     the network's forward (bz_mlp_forward)
  diagnose  moments of every cell and the wall cell's marginal (bz_cell_moments, bz_marginal_v1)
"""
import math

import numpy as np
import torch

from paper_1211_0540_amd import bz

HALF_WIDTH = {8: 4.0, 12: 5.0, 16: 6.0, 20: 6.0, 24: 7.0, 28: 7.5, 32: 8.0}
GATE, S_IN, S_OUT, JUDGE_EVERY = 0.05, 0.05, 1.0, 16
WALL_T = 2.0


def listed():
    return [
        # one cell of Maxwell molecules on the smallest mesh in use: a homogeneous relaxation
        # stepped from a host loop, where launches and latency count
        {"name": "step_n16_1", "path": "step", "mode": "batched_f32", "Ns": "16", "cells": "1", "lam": 0.0,
         "h": 0.05, "start": "mixture", "graph": False},
        # the hard-sphere relaxation of one cell on the finest mesh, replayed as a graph
        {"name": "step_n32_1", "path": "step", "mode": "batched_f32", "Ns": "32", "cells": "1", "lam": 1.0,
         "h": 0.01, "start": "bimaxwellian", "graph": True},
        # the N=32 cells of the uneven batch: the workload of bench.py
        {"name": "step_n32_190", "path": "step", "mode": "batched_f32", "Ns": "32", "cells": "190", "lam": 1.0,
         "h": 0.01, "start": "perturbed", "graph": False},
        # the whole uneven batch, three meshes: the largest call
        {"name": "step_uneven_1024", "path": "step", "mode": "batched_f32", "Ns": "16,24,32",
         "cells": "521,313,190", "lam": 1.0, "h": 0.005, "start": "perturbed", "graph": False},
        # the shock problem: 256 equal cells, Knudsen number 0.1
        {"name": "strang_n24_256", "path": "strang", "mode": "batched_f32", "Ns": "24", "cells": "256", "lam": 1.0,
         "eps": 0.1, "widths": "equal"},
        # the sudden-heating run: 72 cells, narrow at the wall, Knudsen number 1
        {"name": "strang_n24_72", "path": "strang", "mode": "batched_f32", "Ns": "24", "cells": "72", "lam": 1.0,
         "eps": 1.0, "widths": "refined"},
        # FP64 reference values of the 190 cells, and of a ragged small batch by the one-cell path
        {"name": "collide64_n32_190", "path": "collide", "mode": "batched_f64", "Ns": "32", "cells": "190",
         "lam": 1.0, "start": "perturbed"},
        {"name": "plain64_n24_2", "path": "collide", "mode": "plain_f64", "Ns": "24", "cells": "2", "lam": 1.0,
         "start": "perturbed"},
        # the shock problem's collision step with three cells in four served by the network
        {"name": "closure_n24_256", "path": "closure", "mode": "batched_f32", "Ns": "24", "cells": "256",
         "lam": 1.0, "h": 0.5 / 256 / 7.0 / 0.1, "hidden": 1024},
        # the network's training step and its forward at the configured shape
        {"name": "train_512", "path": "train", "Ns": "24", "rows": 512, "hidden": 1024},
        {"name": "serve_256", "path": "serve", "Ns": "24", "rows": 256, "hidden": 1024},
        # what the sudden-heating run records between steps
        {"name": "diagnose_n24_72", "path": "diagnose", "mode": "batched_f32", "Ns": "24", "cells": "72"},
    ]


def draw(rng):
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    path = rng.choice(["step", "step", "step", "strang", "strang", "collide", "collide", "closure", "train", "serve",
                       "diagnose"])
    N = rng.choice([8, 12, 16, 20, 24, 28, 32])
    lam = rng.choice([0.0, 1.0])
    # cells of one mesh that cost no more than the uneven batch
    most = min(1024, 64 * max(1, int(1.8e9 / _pairs(N))))
    if path == "step":
        c = {"path": path, "mode": rng.choice(["batched_f32"] * 5 + ["batched_f64"]), "Ns": str(N), "lam": lam,
             "h": rng.choice([0.002, 0.005, 0.01]), "start": rng.choice(["perturbed", "perturbed", "bimaxwellian"]),
             "graph": rng.random() < 0.3}
        if c["mode"] == "batched_f64":
            most = 64 * max(1, most // 192)
        if rng.random() < 0.3:
            meshes = sorted(rng.sample([8, 12, 16, 20, 24], rng.choice([2, 3])))
            c["Ns"] = ",".join(map(str, meshes))
            c["cells"] = ",".join(str(logint(1, 100)) for _ in meshes)
        else:
            c["cells"] = str(logint(1, most))
        return c
    if path == "strang":
        N = rng.choice([8, 12, 16, 20, 24])
        return {"path": path, "mode": rng.choice(["batched_f32", "batched_f32", "batched_f64"]), "Ns": str(N),
                "cells": str(logint(8, 300)), "lam": lam, "eps": rng.choice([0.1, 1.0]),
                "widths": rng.choice(["equal", "refined"])}
    if path == "collide":
        if rng.random() < 0.3:
            N = rng.choice([8, 12, 16, 20, 24])
            return {"path": path, "mode": "plain_f64", "Ns": str(N), "cells": str(rng.randint(1, 4)), "lam": lam,
                    "start": "perturbed"}
        return {"path": path, "mode": "batched_f64", "Ns": str(N), "lam": lam, "start": "perturbed",
                "cells": str(logint(1, min(300, most)))}
    if path == "closure":
        N = rng.choice([8, 12, 16, 20, 24])
        return {"path": path, "mode": "batched_f32", "Ns": str(N), "cells": str(logint(8, 400)), "lam": lam,
                "h": rng.choice([0.001, 0.003]), "hidden": 32 * logint(1, 32)}
    if path in ("train", "serve"):
        N = rng.choice([8, 12, 16, 20, 24])
        rows = 32 * logint(1, 16) if path == "train" else logint(1, 600)
        return {"path": path, "Ns": str(N), "rows": rows, "hidden": 32 * logint(1, 32)}
    return {"path": path, "mode": "batched_f32", "Ns": str(N), "cells": str(logint(1, 500))}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _pairs(N):
    return (3 * N * N // 4) ** 3


def _ints(text):
    return [int(x) for x in str(text).split(",")]


def _mesh(N):
    L = HALF_WIDTH[N]
    v = (2.0 * L / N) * (torch.arange(N, dtype=torch.float64, device="cuda") - N // 2)
    return v.view(N, 1, 1), v.view(1, N, 1), v.view(1, 1, N)


def _col(x):
    return torch.as_tensor(np.asarray(x, dtype=np.float64), device="cuda").view(-1, 1, 1, 1)


def _maxwellian(N, rho, u, T):
    """rho (2 pi T)^{-3/2} exp(-|v - u|^2 / 2T) for arrays rho, T (n,) and u (n, 3)."""
    V = _mesh(N)
    r2 = sum((V[d] - _col(u[:, d])) ** 2 for d in range(3))
    return _col(rho * (2 * np.pi * T) ** -1.5) * torch.exp(-r2 / _col(2 * T))


def _cells(rng, n, N, start, amp=None):
    """n cells on one mesh, (n, N, N, N) FP64."""
    dv3 = (2.0 * HALF_WIDTH[N] / N) ** 3
    if start == "mixture":      # two counter-streaming Maxwellians, unit mass
        a, one = rng.uniform(0.8, 1.2, n), np.ones(n)
        u = np.stack([a, np.zeros(n), np.zeros(n)], 1)
        f = _maxwellian(N, one, u, one) + _maxwellian(N, one, -u, one)
        return f / (f.sum((1, 2, 3), keepdim=True) * dv3)
    if start == "bimaxwellian":     # three temperatures, unit mass
        V = _mesh(N)
        T = np.stack([rng.uniform(1.5, 2.0, n), rng.uniform(0.5, 0.8, n), rng.uniform(0.5, 0.8, n)], 1)
        f = torch.exp(-sum(V[d] ** 2 / _col(2 * T[:, d]) for d in range(3)))
        return f / (f.sum((1, 2, 3), keepdim=True) * dv3)
    # a Maxwellian with a smooth perturbation of relative size 0.1 (or amp), positive everywhere
    rho, T = rng.uniform(0.5, 2.0, n), rng.uniform(0.5, 2.0, n)
    g = rng.standard_normal((n, 3))
    u = rng.uniform(0.0, 1.5 if N > 8 else 0.5, (n, 1)) * g / np.linalg.norm(g, axis=1, keepdims=True)
    return _perturbed(rng, N, rho, u, T, np.full(n, 0.1) if amp is None else amp)


def _perturbed(rng, N, rho, u, T, amp):
    n, V = len(rho), _mesh(N)
    M = _maxwellian(N, rho, u, T)
    a, kap = rng.standard_normal((n, 6)), rng.uniform(-0.8, 0.8, (n, 6, 3))
    phi = rng.uniform(0.0, 2 * np.pi, (n, 6))
    p = torch.zeros_like(M)
    for i in range(6):
        arg = sum(_col(kap[:, i, d] / np.sqrt(T)) * (V[d] - _col(u[:, d])) for d in range(3)) + _col(phi[:, i])
        p += _col(a[:, i]) * torch.cos(arg)
    p *= ((M ** 2).sum((1, 2, 3), keepdim=True) / ((M * p) ** 2).sum((1, 2, 3), keepdim=True)).sqrt()
    p *= _col(amp)
    p *= (0.9 / (-p).amax((1, 2, 3), keepdim=True).clamp_min(0.9))
    return M * (1.0 + p)


def _heated(rng, n, N):
    """Gas at rest with a layer heated by the wall at x = 0, in x order."""
    x = (np.arange(n) + 0.5) / n
    w = rng.uniform(0.3, 0.6) * np.exp(-x / rng.uniform(0.05, 0.15))
    one, zero = np.ones(n), np.zeros(n)
    hot = _maxwellian(N, one, np.stack([zero + rng.uniform(0.05, 0.15), zero, zero], 1), 1.8 * one)
    f = _col(1 - w) * _maxwellian(N, one, np.zeros((n, 3)), one) + _col(w) * hot
    return f * (1 + 0.05 * _col(w) * torch.cos(_mesh(N)[0] + rng.uniform(0, 6)))


def _near_equilibrium(rng, n, N):
    """The first quarter of the cells away from equilibrium, the others within the gate."""
    q = n // 4
    amp = np.concatenate([rng.uniform(0.1, 0.3, q), np.exp(rng.uniform(np.log(1e-4), np.log(0.02), n - q))])
    x = np.arange(n) / n
    u = np.stack([0.2 * np.exp(-4 * x), 0 * x, 0 * x], 1)
    return _perturbed(rng, N, 1 + 0.1 * np.exp(-4 * x), u, 1 + 0.4 * np.exp(-4 * x), amp)


def _state_of(case, seed):
    """Input cells of a collision case: one (n, N, N, N) tensor per mesh, and the mesh of every cell."""
    rng = np.random.default_rng(seed)
    Ns, counts = _ints(case["Ns"]), _ints(case["cells"])
    if case["path"] in ("strang", "diagnose"):
        parts = [_heated(rng, counts[0], Ns[0])]
    elif case["path"] == "closure":
        parts = [_near_equilibrium(rng, counts[0], Ns[0])]
    else:
        parts = [_cells(rng, n, N, case["start"]) for N, n in zip(Ns, counts)]
    mesh_of = np.repeat(np.arange(len(Ns)), counts)
    if len(Ns) > 1:
        rng.shuffle(mesh_of)
    return Ns, parts, mesh_of


def _flat(parts, mesh_of):
    """Cells in batch order, back to back."""
    if len(parts) == 1:
        return parts[0].reshape(-1).clone()
    at = [0] * len(parts)
    out = []
    for m in mesh_of:
        out.append(parts[m][at[m]].reshape(-1))
        at[m] += 1
    return torch.cat(out)


def _widths(case):
    n = _ints(case["cells"])[0]
    if case["widths"] == "equal":
        return np.full(n, 1.0 / n)
    w = np.minimum(0.125 * 1.1 ** np.maximum(np.arange(n) - 8, 0), 0.5)     # eps/8 at the wall, eps/2 inside
    return w


def _network(seed, N, hidden):
    """Master weights [W1 b1 W2 b2 W3 b3], FP32 on the host."""
    gen = torch.Generator().manual_seed(int(seed))
    M, parts = N ** 3, []
    for o, i in ((hidden, M), (hidden, hidden), (M, hidden)):
        s = 1.0 / math.sqrt(i)
        parts += [(torch.rand(o * i, generator=gen) * 2 - 1) * s, (torch.rand(o, generator=gen) * 2 - 1) * s]
    return torch.cat(parts)


def _rows(seed, N, rows):
    """Network inputs (BF16 of unit RMS) and targets of order one."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    M = N ** 3
    x = torch.randn(rows, M, generator=gen, device="cuda").to(torch.bfloat16)
    return x, 0.5 * torch.randn(rows, M, generator=gen, device="cuda")


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
_WEIGHTS = {}   # the weight streams of the meshes in use, kept as a program keeps them


class _State:
    """What a program holds; its handles are given back with it."""

    def __init__(self):
        self.graph = self.transport = self.net = None

    def __del__(self):
        if self.graph:
            bz.bz_graph_free(self.graph)
        if self.transport:
            bz.bz_transport_free(self.transport)
        if self.net:
            bz.bz_mlp_free(self.net)


def _collision(case, Ns, mesh_of, fine_split=False):
    if sum(b.numel() for b in _WEIGHTS.values()) > 12e9:
        _WEIGHTS.clear()
    meshes = [(N, HALF_WIDTH[N], case.get("lam", 1.0)) for N in Ns]
    return bz.Collision(meshes, mesh_of, case["mode"], weights_cache=_WEIGHTS, fine_split=fine_split)


def prepare(case, seed):
    s = _State()
    s.path = case["path"]
    N = _ints(case["Ns"])[0]
    if s.path in ("train", "serve", "closure"):
        s.net = bz.bz_mlp_create(N ** 3, case["hidden"], N ** 3)
        s.params = torch.zeros(bz.bz_mlp_param_bytes(s.net), dtype=torch.uint8, device="cuda")
        bz.bz_mlp_set_params(s.net, s.params, _network(seed, N, case["hidden"]).numpy())
    if s.path in ("train", "serve"):
        s.rows, s.n = case["rows"], bz.bz_mlp_param_count(s.net)
        x, s.y = _rows(seed, N, s.rows)
        s.x = x.view(torch.int16)
        s.work = torch.zeros(bz.bz_mlp_workspace_bytes(s.net, s.rows), dtype=torch.uint8, device="cuda")
        s.grad = torch.zeros(s.n, dtype=torch.float32, device="cuda")
        s.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        s.weights = s.params[:4 * s.n].view(torch.float32)
        s.out = torch.zeros(s.rows, N ** 3, dtype=torch.float32, device="cuda")
        s.step = 0
        return s
    Ns, parts, mesh_of = _state_of(case, seed)
    s.f = _flat(parts, mesh_of)
    s.col = _collision(case, Ns, mesh_of, fine_split=s.path == "closure")
    if s.path == "step":
        s.h = case["h"]
        if case["graph"]:
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.current_stream())
            s.graph = bz.bz_graph_capture_step(s.col.batch, s.f, s.h, s.col.work, stream)
    elif s.path == "strang":
        w = _widths(case)
        s.transport = bz.bz_transport_create_ex(s.col.grids[0], w, WALL_T, 1.0, 0.0, 1.0)
        s.dt, s.eps = 0.5 * float(w.min()) / HALF_WIDTH[N], case["eps"]
        need = bz.bz_strang_workspace_bytes(s.col.batch, s.transport)
        s.col.work = torch.zeros(need, dtype=torch.uint8, device="cuda")
    elif s.path == "collide":
        s.q = torch.zeros_like(s.f)
    elif s.path == "closure":
        # a judge that does not fail: what a trained network meets
        s.h, s.f0 = case["h"], s.f.clone()
        s.desc = bz.closure_desc(s.net, s.params, GATE, S_IN, S_OUT, JUDGE_EVERY, judge_tol=1e30)
        s.work = torch.zeros(bz.bz_closure_workspace_bytes(s.col.batch, s.desc), dtype=torch.uint8, device="cuda")
    else:
        s.mom = torch.zeros(5 * len(mesh_of), dtype=torch.float64, device="cuda")
        s.marg = torch.zeros(N, dtype=torch.float64, device="cuda")
    return s


def run(s):
    if s.path == "step":
        if s.graph:
            bz.bz_graph_launch(s.graph)
        else:
            s.col.step(s.f, s.h)
        return s.f
    if s.path == "strang":
        return s.col.strang_step(s.transport, s.dt, s.eps, s.f)
    if s.path == "collide":
        return s.col.project(s.col.collide(s.f, out=s.q))
    if s.path == "closure":
        # from the same state each time: the share of served cells stays what it is
        s.f.copy_(s.f0)
        bz.bz_closure_step(s.col.batch, s.desc, s.f, s.h, s.work)
        return s.f
    if s.path == "train":
        s.step += 1
        bz.bz_mlp_backward(s.net, s.params, s.x, s.y, s.rows, s.grad, s.loss, s.work)
        bz.bz_mlp_adam(s.net, s.params, s.grad, s.step, 1e-4)
        return {"grad": s.grad, "loss": s.loss, "weights": s.weights}
    if s.path == "serve":
        bz.bz_mlp_forward(s.net, s.params, s.x, s.rows, s.out, s.work)
        return s.out
    bz.bz_cell_moments(s.col.batch, s.f, s.mom)
    bz.bz_marginal_v1(s.col.batch, s.f, 0, s.marg)
    return {"moments": s.mom, "marginal": s.marg}


def work(case):
    Ns = _ints(case["Ns"])
    if case["path"] in ("train", "serve"):
        M, H, B = Ns[0] ** 3, case["hidden"], case["rows"]
        weights = 2 * M * H + H * H
        if case["path"] == "serve":
            return {"bytes": 2 * weights + 2 * B * M + 4 * B * M, "flops": 2.0 * B * weights}
        # forward and weight gradients over all layers, input gradients of layers 2 and 3; Adam
        # reads and writes the master and both moments and writes the gradient
        return {"bytes": 28 * weights + 6 * B * M, "flops": 2.0 * B * (2 * weights + M * H + H * H)}
    counts = _ints(case["cells"])
    elems = sum(n * N ** 3 for N, n in zip(Ns, counts))
    if case["path"] == "diagnose":
        return {"bytes": 8 * elems, "flops": 10 * elems}
    # a pair once for each half of the outputs: 10 operations, its weight read once a mesh
    evals = 1 if case["path"] == "collide" else 2
    size = 4 if case["mode"].endswith("f32") else 8
    share = 0.25 if case["path"] == "closure" else 1.0      # the cells that are not served
    pairs = sum(n * _pairs(N) / 4 for N, n in zip(Ns, counts))
    return {"bytes": 16 * elems + size * sum(_pairs(N) / 4 for N in Ns), "flops": evals * share * 10 * pairs}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _table(N, lam):
    """T(p, q) = int_0^1 s^{lam+2} sinc(pi s sqrt(p)/2) sinc(pi s sqrt(q)/2) ds, lam = 0 or 1, in closed form."""
    a = (np.pi / 2 * np.sqrt(np.arange(3 * N * N // 4 + 1)))[:, None]
    b = (np.pi / 2 * np.sqrt(np.arange(3 * N * N + 1)))[None, :]

    def F(x):
        y = np.where(x == 0, 1.0, x)
        s = np.sin(y) / y
        if lam == 0:
            return np.where(x == 0, 1.0, s)
        return np.where(x == 0, 0.5, s - 2 * np.sin(y / 2) ** 2 / (y * y))

    with np.errstate(divide="ignore", invalid="ignore"):
        T = (F(a - b) - F(a + b)) / (2 * a * b)

    def edge(c):
        c = np.where(c == 0, 1.0, c)
        if lam == 0:
            return (np.sin(c) - c * np.cos(c)) / c ** 3
        return (-np.cos(c) / c + 2 * np.sin(c) / c ** 2 - 4 * np.sin(c / 2) ** 2 / c ** 3) / c

    T[0], T[:, 0] = edge(b[0]), edge(a[:, 0])
    T[0, 0] = 1.0 / (lam + 3)
    return torch.as_tensor(T, device="cuda")


def _transform(x, N, sign):
    """Centred discrete transform over the last three axes of (n, N, N, N)."""
    k = torch.arange(N, dtype=torch.float64, device="cuda") - N // 2
    E = torch.exp(sign * 2j * np.pi / N * k[:, None] * k[None, :])
    for _ in range(3):      # each turn transforms the last axis and brings it to the front
        x = (x.reshape(-1, N) @ E).reshape(-1, N, N, N).permute(0, 3, 1, 2).contiguous()
    return x


def _collide(f, lam, table):
    """Q (projected) of cells f (n, N, N, N): the trapezoid sum, pair by pair."""
    n, N = f.shape[0], f.shape[1]
    h, L, dev = N // 2, HALF_WIDTH[N], f.device
    dv, dz = 2 * L / N, np.pi / L
    fh = _transform(f.to(torch.complex128), N, -1) * ((2 * np.pi) ** -1.5 * dv ** 3)
    s = 4 * np.pi * (2 * np.pi) ** -1.5 * L ** (lam + 3) * dz ** 3
    # reversed axes: index j of a partner is N - 1 - j; zeros where it leaves the mesh on axis 3
    rev = torch.nn.functional.pad(torch.view_as_real(fh.flip(1, 2, 3)), (0, 0, h, h - 1))
    rev = torch.view_as_complex(rev.contiguous())
    i = torch.arange(N, device=dev)
    out = torch.zeros_like(fh)
    for k1 in range(N):
        for k2 in range(N):
            a0, a1 = max(0, k1 - h + 1), min(N - 1, k1 + h)
            b0, b1 = max(0, k2 - h + 1), min(N - 1, k2 + h)
            m1, m2 = i[a0:a1 + 1].view(-1, 1, 1, 1), i[b0:b1 + 1].view(1, -1, 1, 1)
            k3, m3 = (N - 1 - i).view(1, 1, -1, 1), i.view(1, 1, 1, -1)     # window w holds k3 = N - 1 - w
            na = (k1 - h) ** 2 + (k2 - h) ** 2 + (k3 - h) ** 2
            nb = (2 * m1 - k1 - h) ** 2 + (2 * m2 - k2 - h) ** 2 + (2 * m3 - k3 - h) ** 2
            nc = (m1 - h) ** 2 + (m2 - h) ** 2 + (m3 - h) ** 2
            W = s * (table[na, nb.clamp_max(3 * N * N)] - table[0][4 * nc])
            for c in range(0, n, max(1, 40_000_000 // W.numel())):
                e = c + max(1, 40_000_000 // W.numel())
                x = fh[c:e, a0:a1 + 1, b0:b1 + 1].unsqueeze(3)
                # partner index of m1 on the reversed axis: m1 - k1 + h - 1
                y = rev[c:e, a0 - k1 + h - 1:a1 - k1 + h, b0 - k2 + h - 1:b1 - k2 + h].unfold(3, N, 1)
                out[c:e, k1, k2] = ((y * W) * x).sum((1, 2, 4)).flip(1)
    qt = _transform(out, N, +1).real * ((2 * np.pi) ** -1.5 * dz ** 3)
    V = _mesh(N)
    one = torch.ones(N, N, N, dtype=torch.float64, device=dev)
    C = torch.stack([one, V[0] * one, V[1] * one, V[2] * one, (V[0] ** 2 + V[1] ** 2 + V[2] ** 2) * one]).view(5, -1)
    q = qt.reshape(n, -1)
    for _ in range(2):
        q = q - torch.linalg.solve((C @ C.T).cpu(), (C @ q.T).cpu()).to(dev).T @ C
    return q.view_as(qt)


def _heun(f, h, Q):
    fs = f + h * Q(f)
    return 0.5 * (f + fs + h * Q(fs))


def _transport(f, w, dt):
    """Heun step of df/dt + v1 df/dx = 0: minmod slopes, diffuse wall on the left, gas at rest on the right."""
    n, N = f.shape[0], f.shape[1]
    v, one = _mesh(N)[0], np.ones(1)
    wall = _maxwellian(N, one, np.zeros((1, 3)), WALL_T * one)
    far = _maxwellian(N, one, np.zeros((1, 3)), one)
    we = torch.cat([w[:1], w[:1], w, w[-1:], w[-1:]]).view(-1, 1, 1, 1)
    gap = 0.5 * (we[1:] + we[:-1])

    def rhs(g):
        e = torch.cat([g[:1], g[:1], g, far, far])
        s = (e[1:] - e[:-1]) / gap
        a, b = s[:-1], s[1:]
        sl = torch.where(a * b > 0, torch.where(a > 0, torch.minimum(a, b), torch.maximum(a, b)), torch.zeros_like(a))
        c, wc = e[1:-1], we[1:-1]      # cells -1 .. n
        left = v * (c[:-1] + 0.5 * wc[:-1] * sl[:-1])
        right = v * (c[1:] - 0.5 * wc[1:] * sl[1:])
        F = torch.where(v >= 0, left, right)     # faces -1/2 .. n - 1/2
        sigma = -(v.clamp_max(0) * g[0]).sum() / (v.clamp_min(0) * wall[0]).sum()
        F[0] = torch.where(v > 0, v * sigma * wall[0], v * g[0])
        return -(F[1:] - F[:-1]) / we[2:-2]

    fs = f + dt * rhs(f)
    return 0.5 * (f + fs + dt * rhs(fs))


def _layers(seed, N, hidden):
    """The network's weights as its products take them: BF16 matrices, FP32 biases."""
    v, o, out = _network(seed, N, hidden).cuda(), 0, []
    for a, b in ((hidden, N ** 3), (hidden, hidden), (N ** 3, hidden)):
        out.append(v[o:o + a * b].view(a, b).to(torch.bfloat16).double())
        out.append(v[o + a * b:o + a * b + a].double())
        o += a * b + a
    return out


def _gelu(z):
    return 0.5 * z * (1 + torch.erf(z / math.sqrt(2)))


def _forward(p, x):
    z1 = x @ p[0].T + p[1]
    z2 = _gelu(z1) @ p[2].T + p[3]
    return z1, z2, _gelu(z2) @ p[4].T + p[5]


def _closure_q(f, case, p, table, phase):
    n, N = f.shape[0], f.shape[1]
    dv3, V = (2 * HALF_WIDTH[N] / N) ** 3, _mesh(N)

    def mean(w):
        return (f * w).sum((1, 2, 3)) * dv3

    rho = mean(1.0)
    u = [mean(V[d]) / rho for d in range(3)]
    T = (mean(V[0] ** 2 + V[1] ** 2 + V[2] ** 2) / rho - sum(a * a for a in u)) / 3
    M = _maxwellian(N, rho.cpu().numpy(), torch.stack(u, 1).cpu().numpy(), T.cpu().numpy())
    D = (f - M).reshape(n, -1)
    dn, mn = D.norm(dim=1), M.reshape(n, -1).norm(dim=1)
    d = dn / mn
    x = D * (math.sqrt(N ** 3) / dn)[:, None]
    x[:, 0] = d / S_IN
    q = ((rho * dn * S_OUT)[:, None] * _forward(p, x.to(torch.bfloat16).double())[2]).view_as(f)
    judged = torch.arange(n, device="cuda") // 64 % JUDGE_EVERY == phase % JUDGE_EVERY
    need = torch.nonzero((d >= GATE) | judged).flatten()
    conv = _collide(f[need], case["lam"], table)
    V1 = torch.ones(N, N, N, dtype=torch.float64, device="cuda")
    C = torch.stack([V1, V[0] * V1, V[1] * V1, V[2] * V1, (V[0] ** 2 + V[1] ** 2 + V[2] ** 2) * V1]).view(5, -1)
    q = q.reshape(n, -1)
    for _ in range(2):
        q = q - torch.linalg.solve((C @ C.T).cpu(), (C @ q.T).cpu()).cuda().T @ C
    q = q.view_as(f)
    q[need] = conv
    return q


def exact(case, seed):
    Ns = _ints(case["Ns"])
    N = Ns[0]
    if case["path"] in ("train", "serve"):
        p = _layers(seed, N, case["hidden"])
        x, y = _rows(seed, N, case["rows"])
        x = x.double()
        z1, z2, out = _forward(p, x)
        if case["path"] == "serve":
            return out
        d = 2 * (out - y) / y.numel()

        def slope(z):
            return 0.5 * (1 + torch.erf(z / math.sqrt(2))) + z * torch.exp(-z * z / 2) / math.sqrt(2 * math.pi)

        d2 = (d @ p[4]) * slope(z2)
        d1 = (d2 @ p[2]) * slope(z1)
        g = torch.cat([(d1.T @ x).flatten(), d1.sum(0), (d2.T @ _gelu(z1)).flatten(), d2.sum(0),
                       (d.T @ _gelu(z2)).flatten(), d.sum(0)])
        # Adam's first step is g / (|g| + eps), a sign, which 64 bits of the inputs do not fix
        return {"grad": g, "loss": ((out - y) ** 2).mean().reshape(1), "weights": None}
    _, parts, mesh_of = _state_of(case, seed)
    if case["path"] == "diagnose":
        f, V = parts[0], _mesh(N)
        dv = 2 * HALF_WIDTH[N] / N
        rho = f.sum((1, 2, 3))
        u = [(f * V[d]).sum((1, 2, 3)) / rho for d in range(3)]
        T = (sum((V[d] - u[d].view(-1, 1, 1, 1)) ** 2 for d in range(3)) * f).sum((1, 2, 3)) / (3 * rho)
        return {"moments": torch.stack([rho * dv ** 3, *u, T], 1).flatten(), "marginal": f[0].sum((1, 2)) * dv ** 2}
    lam = case["lam"]
    done = []
    for M, f in zip(Ns, parts):
        table = _table(M, lam)
        if case["path"] == "step":
            done.append(_heun(f, case["h"], lambda g: _collide(g, lam, table)))
        elif case["path"] == "collide":
            done.append(_collide(f, lam, table))
        elif case["path"] == "strang":
            w = torch.as_tensor(_widths(case), device="cuda")
            dt = 0.5 * float(w.min()) / HALF_WIDTH[M]
            f = _transport(f, w, 0.5 * dt)
            f = _heun(f, dt / case["eps"], lambda g: _collide(g, lam, table))
            done.append(_transport(f, w, 0.5 * dt))
        else:
            p = _layers(seed, M, case["hidden"])
            phase = iter(range(2))
            done.append(_heun(f, case["h"], lambda g: _closure_q(g, case, p, table, next(phase))))
    return _flat(done, mesh_of)
