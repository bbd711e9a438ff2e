"""Performance cases of the solver: what users have it do, through the public
entry points, from one launch-bound system to gigabyte solves.

listed() names the fixed cases, draw(rng) makes another one of the same
ranges; prepare(case, seed) builds what a program holds before the call (the
plan and the device inputs), run(state) is one pass through the entry points,
work(case) the bytes and operations of a pass, and exact(case, seed) the same
outputs in plain 64-bit torch.

Kinds:
  series     M right-hand sides sharing one matrix (Plan): the single systems
             of the headline, series, and the short lines of a 3D array;
             quasi-Toeplitz ends, gradients and the three precisions optional
  autograd   one training step through TridiagToeplitzSolve (values in t)
  varlen     systems of their own sizes and matrices (VarlenPlan): the modes
             of a separation of variables, or a differentiable batch
  general    M right-hand sides of one per-row matrix (GeneralPlan)
  strided    systems along a slow axis (StridedPlan)
  poisson2d, poisson3d   the end-to-end Poisson solves
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1002_2469_amd as tdt

DEV = "cuda"


def listed() -> list:
    return [
        # the smallest call in earnest: one system of 65536 rows, bound by
        # launches and latency
        dict(name="single_65536_f64", kind="series", n=65536, m=1, dtype="f64", quasi=False,
             grad=False, ratio=2.0, shape=0),
        # the headline: one system of 2^26 rows, float sweeps refined to
        # double, in the work shape the autotuner picks for it
        dict(name="single_2e26_refine", kind="series", n=1 << 26, m=1, dtype="f32_refine",
             quasi=False, grad=False, ratio=1.25, shape=2),
        # an ordinary float series whose size is no multiple of anything
        dict(name="series_512x30011_f32", kind="series", n=30011, m=512, dtype="f32",
             quasi=False, grad=False, ratio=1.5, shape=0),
        # the contiguous lines of a 255^3 grid: many short systems, solved
        # along the last dimension of an array
        dict(name="lines_65025x255_f64", kind="series", n=255, m=255 * 255, dtype="f64",
             quasi=False, grad=False, ratio=1.5, shape=0),
        # the modes of a separation of variables (sizes 256 to 65536), with
        # the autotuner's choice for them
        dict(name="sov_2048_f64", kind="varlen", s=2048, n_min=256, n_max=65536, layout=0,
             matrices="sov", dtype="f64", quasi=False, grad=False, shape=2, whole=0),
        # Neumann ends, refinement, forward and adjoint (default options)
        dict(name="neumann_1000_refine_grad", kind="varlen", s=1000, n_min=100, n_max=20000,
             layout=1, matrices="sov", dtype="f32_refine", quasi=True, grad=True, shape=0,
             whole=8),
        # a differentiable batch: forward and adjoint of 1024 systems
        dict(name="diff_1024x16384_f64_grad", kind="varlen", s=1024, n_min=16384, n_max=16384,
             layout=0, matrices="dominant", dtype="f64", quasi=False, grad=True, shape=2,
             whole=16),
        # a variable-coefficient operator, forward and adjoint with the
        # gradients of its entries, ragged size
        dict(name="general_24x500009_f64_grad", kind="general", n=500009, m=24, dtype="f64",
             grad=True),
        # line solves along a slow axis, longer than one column
        dict(name="strided_4x2000x1023", kind="strided", n=2000, m=1023, nb=4),
        # end to end Poisson solves: the 2^13 grid, an ordinary grid of 1000
        # by 1500 intervals, and the 3D benchmark grid
        dict(name="poisson2d_8191", kind="poisson2d", nx=8191, ny=8191),
        dict(name="poisson2d_999x1499", kind="poisson2d", nx=999, ny=1499),
        dict(name="poisson3d_511", kind="poisson3d", nx=511, ny=511, nz=511),
    ]


def _logint(rng, lo, hi) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["series", "series", "series", "autograd", "varlen", "varlen", "general",
                       "strided", "poisson2d", "poisson2d", "poisson3d"])
    if kind in ("series", "autograd"):
        n = _logint(rng, 64, 1 << 26)
        if rng.random() < 0.25:
            n = max(64, n // 4096 * 4096)
        total = _logint(rng, max(n, 1 << 14), max(n, 1 << 25))
        grad = kind == "autograd" or rng.random() < 0.3
        return dict(kind=kind, n=n, m=max(1, min(total // n, 400000)),
                    dtype=rng.choice(["f64", "f64", "f32", "f32_refine"]),
                    quasi=rng.random() < 0.25, grad=grad, ratio=rng.uniform(1.1, 3.0),
                    shape=0 if kind == "autograd" else rng.choice([0, 0, 1, 2]))
    if kind == "varlen":
        a, b = _logint(rng, 16, 65536), _logint(rng, 16, 65536)
        total = _logint(rng, 1 << 16, 1 << 24)
        lo, hi = min(a, b), max(a, b)
        return dict(kind=kind, s=max(1, min(total // hi, 20000)), n_min=lo, n_max=hi,
                    layout=rng.randrange(1 << 16), matrices=rng.choice(["sov", "dominant"]),
                    dtype=rng.choice(["f64", "f64", "f32", "f32_refine"]),
                    quasi=rng.random() < 0.3, grad=rng.random() < 0.4,
                    shape=rng.choice([0, 0, 1, 2]), whole=rng.choice([8, 8, 0, 16]))
    if kind == "general":
        n = _logint(rng, 1000, 1 << 20)
        if rng.random() < 0.3:
            n = max(4096, n // 4096 * 4096)
        total = _logint(rng, max(n, 1 << 15), 1 << 25)
        return dict(kind=kind, n=n, m=max(1, min(total // n, 4096)),
                    dtype=rng.choice(["f64", "f32"]), grad=rng.random() < 0.4)
    if kind == "strided":
        n = _logint(rng, 16, 20000)
        total = _logint(rng, max(64 * n, 1 << 16), max(64 * n, 1 << 25))
        m = min(_logint(rng, 16, 4000), max(16, total // n))
        return dict(kind=kind, n=n, m=m, nb=max(1, min(total // (n * m), 1024)))
    if kind == "poisson2d":
        nx = (1 << rng.randrange(7, 14)) - 1 if rng.random() < 0.5 else _logint(rng, 20, 6000)
        return dict(kind=kind, nx=nx, ny=min(_logint(rng, 20, 8191), (1 << 25) // nx))
    nx = (1 << rng.randrange(7, 10)) - 1 if rng.random() < 0.5 else _logint(rng, 20, 500)
    ny = _logint(rng, 20, 500)
    return dict(kind=kind, nx=nx, ny=ny, nz=max(10, min(_logint(rng, 20, 500),
                                                        (1 << 25) // (nx * ny))))


# --------------------------------------------------------------------------
# inputs: host matrices from numpy, device arrays from torch, by the seed
# --------------------------------------------------------------------------
def _normal(seed, stream, shape, dtype=torch.float64):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + stream)
    return torch.randn(shape, dtype=dtype, device=DEV, generator=g)


def _io(dtype):
    return torch.float32 if dtype == "f32" else torch.float64


def _series_matrix(case, seed):
    """(t_-1, t_0, t_1, psi, chi): an unsymmetric stencil of the case's
    dominance ratio; the corners are a mirrored ghost value's."""
    rng = np.random.default_rng(seed)
    s = rng.uniform(0.9, 1.1)
    a, c = -0.9 * s, -1.1 * s
    return a, case["ratio"] * (abs(a) + abs(c)), c, 0.4 * s, 0.5 * s


def _varlen_system(case, seed):
    """offsets and per-system (t_-1, t_0, t_1)."""
    s = case["s"]
    rng = np.random.default_rng(case["layout"])
    sizes = np.rint(np.exp(rng.uniform(math.log(case["n_min"]), math.log(case["n_max"]), s)))
    off = np.zeros(s + 1, dtype=np.int64)
    np.cumsum(np.maximum(sizes.astype(np.int64), 3), out=off[1:])
    rng = np.random.default_rng(seed)
    if case["matrices"] == "sov":
        r = rng.uniform(0.5, 2.0, s)
        k = np.arange(1, s + 1, dtype=np.float64)
        t0 = -(2.0 + 4.0 * r * r * np.sin(k * math.pi / (2.0 * (s + 1))) ** 2)
        # float solves leave out the modes that float cannot resolve, Neumann
        # problems carry a small reaction term (the lowest mode is singular)
        t0 -= 0.02 if case["dtype"] != "f64" else (1e-4 if case["quasi"] else 0.0)
        return off, np.ones(s), t0, np.ones(s)
    return off, rng.uniform(-1.0, -0.5, s), rng.uniform(2.5, 4.0, s), rng.uniform(-1.0, -0.5, s)


def _general_rows(case, seed):
    """Rows of a variable-coefficient diffusion-reaction operator."""
    n = case["n"]
    rng = np.random.default_rng(seed)
    x = (np.arange(n + 1) + 0.5) / (n + 1)
    kap = np.exp(0.5 * np.sin(2.0 * math.pi * x) + 0.3 * rng.uniform(-1.0, 1.0, n + 1))
    e = rng.uniform(-0.3, 0.3, n)
    a, c = -kap[:-1] * (1.0 + e), -kap[1:] * (1.0 - e)
    return a, rng.uniform(1.1, 1.6, n) * (np.abs(a) + np.abs(c)), c


def _strided_matrix(case, seed):
    """One class per system: the modes' lines of a Poisson problem."""
    m = case["m"]
    r = np.random.default_rng(seed).uniform(0.8, 1.25)
    k = np.arange(1, m + 1, dtype=np.float64)
    return -1.0, 2.0 + 4.0 * r * np.sin(k * math.pi / (2.0 * (m + 1))) ** 2, -1.0


def _inputs(case, seed):
    kind = case["kind"]
    if kind in ("series", "autograd", "general"):
        shape = (case["m"], case["n"])
    elif kind == "varlen":
        shape = (int(_varlen_system(case, seed)[0][-1]),)
    elif kind == "strided":
        shape = (case["nb"], case["n"], case["m"])
    elif kind == "poisson2d":
        shape = (case["ny"], case["nx"])
    else:
        shape = (case["nz"], case["ny"], case["nx"])
    dt = _io(case.get("dtype", "f64"))
    F = _normal(seed, 1, shape, dt)
    W = _normal(seed, 2, shape, dt) if case.get("grad") else None
    return F, W


def prepare(case, seed):
    kind = case["kind"]
    F, W = _inputs(case, seed)
    st = dict(kind=kind, F=F, W=W)
    if kind in ("series", "autograd"):
        a, b, c, psi, chi = _series_matrix(case, seed)
        q = dict(psi=psi, chi=chi) if case["quasi"] else {}
        if kind == "autograd":
            st["dtype"] = case["dtype"]
            st["t"] = torch.tensor([a, b, c] + ([psi, chi] if q else []), dtype=torch.float64,
                                   requires_grad=True)
            st["F"] = F.requires_grad_(True)
            return st
        st["plan"] = tdt.Plan(a, b, c, case["n"], case["dtype"], **q)
        if case["shape"]:
            st["plan"].set_option("shape", case["shape"])
    elif kind == "varlen":
        off, tm1, t0, t1 = _varlen_system(case, seed)
        q = dict(psi=tm1, chi=t1) if case["quasi"] else {}
        st["plan"] = tdt.VarlenPlan(off, tm1, t0, t1, case["dtype"], **q)
        if case["shape"]:
            st["plan"].set_option("shape", case["shape"])
        if case["whole"] != 8:
            st["plan"].set_option("whole_max_tiles", case["whole"])
    elif kind == "general":
        st["plan"] = tdt.GeneralPlan(*_general_rows(case, seed), case["dtype"])
    elif kind == "strided":
        st["plan"] = tdt.StridedPlan(case["n"], *_strided_matrix(case, seed))
    elif kind == "poisson2d":
        st["plan"] = tdt.Poisson2D(case["nx"], case["ny"], 1.0 / (case["nx"] + 1),
                                   1.0 / (case["ny"] + 1))
    else:
        st["plan"] = tdt.Poisson3D(case["nx"], case["ny"], case["nz"], 1.0 / (case["nx"] + 1),
                                   1.0 / (case["ny"] + 1), 1.0 / (case["nz"] + 1))
    return st


def run(st):
    if st["kind"] == "autograd":
        F, t = st["F"], st["t"]
        X = tdt.TridiagToeplitzSolve.apply(F, t, st["dtype"])
        gF, gt = torch.autograd.grad(X, (F, t), st["W"])
        return X.detach(), gF, gt
    X = st["plan"].solve(st["F"])
    if st["W"] is None:
        return X
    gF, g = st["plan"].backward(st["W"], X)
    return X, gF, g


def work(case) -> dict:
    kind = case["kind"]
    size = 4 if case.get("dtype") == "f32" else 8
    if kind in ("series", "autograd", "general"):
        u = case["n"] * case["m"]
    elif kind == "varlen":
        u = int(_varlen_system(case, 0)[0][-1])
    elif kind == "strided":
        u = case["n"] * case["m"] * case["nb"]
    elif kind == "poisson2d":
        u = case["nx"] * case["ny"]
    else:
        u = case["nx"] * case["ny"] * case["nz"]
    # a solve reads F and writes X; its adjoint reads gX and X, writes gF
    nbytes = u * size * (5 if case.get("grad") else 2)
    flops = u * (22 if case.get("grad") else 8)   # two sweeps; the gradients' products
    if kind == "general":   # the matrix, and its entries' gradients
        nbytes += case["n"] * (3 * size + (24 if case["grad"] else 0))
    if kind in ("poisson2d", "poisson3d"):
        # two real transforms of length nx + 1 per row; ADI half-steps in 3D
        flops += u * 5 * math.log2(case["nx"] + 1)
    if kind == "poisson3d":
        flops += u * 12 * 2 * 10
    return dict(bytes=int(nbytes), flops=int(flops))


# --------------------------------------------------------------------------
# exact: plain 64-bit torch
# --------------------------------------------------------------------------
def _shift(v, d):
    """v moved by d entries, zeros moved in (d > 0: out[i] = v[i - d])."""
    out = torch.zeros_like(v)
    if d > 0:
        out[d:] = v[:-d]
    else:
        out[:d] = v[-d:]
    return out


def _pcr(a, b, c, f, longest):
    """Parallel cyclic reduction of the tridiagonal rows (a, b, c); a and c
    are 0 at the ends of every system."""
    d = 1
    while d < longest:
        k1 = a / _shift(b, d).masked_fill_(a == 0, 1.0)
        k2 = c / _shift(b, -d).masked_fill_(c == 0, 1.0)
        f = f - k1 * _shift(f, d) - k2 * _shift(f, -d)
        b = b - k1 * _shift(c, d) - k2 * _shift(a, -d)
        a, c = -k1 * _shift(a, d), -k2 * _shift(c, -d)
        del k1, k2
        d *= 2
        if not (bool(a.any()) or bool(c.any())):
            break
    return f / b


def _two_prod(x, y):
    """x y as a sum of two doubles (Dekker's splitting)."""
    p = x * y
    t = 134217729.0 * x
    xh = t - (t - x)
    t = 134217729.0 * y
    yh = t - (t - y)
    xl, yl = x - xh, y - yh
    return p, ((xh * yh - p) + xh * yl + xl * yh) + xl * yl


def _solve_flat(a, b, c, f, longest):
    """PCR, then one refinement with the residual in twice the precision."""
    x = _pcr(a, b, c, f, longest)
    s, e = f, torch.zeros_like(f)
    for m, v in ((b, x), (a, _shift(x, 1)), (c, _shift(x, -1))):
        p, q = _two_prod(m, v)
        t = s - p
        z = t - s
        e = e + ((s - (t - z)) + (-p - z)) - q
        s = t
    return x + _pcr(a, b, c, s + e, longest)


def _flat_rows(case, seed):
    """(a, b, c) of the whole case as one tridiagonal matrix without coupling
    between systems, the index of every row's system, and the longest one."""
    kind = case["kind"]
    dev = dict(dtype=torch.float64, device=DEV)
    if kind == "general":
        n, m = case["n"], case["m"]
        a, b, c = (torch.tensor(v, **dev) for v in _general_rows(case, seed))
        a[0], c[-1] = 0.0, 0.0
        return a.repeat(m), b.repeat(m), c.repeat(m), None, n
    if kind == "varlen":
        off, tm1, t0, t1 = _varlen_system(case, seed)
        psi, chi = (tm1, t1) if case["quasi"] else (0.0 * tm1, 0.0 * t1)
    else:
        v = _series_matrix(case, seed)
        off = np.arange(case["m"] + 1, dtype=np.int64) * case["n"]
        tm1, t0, t1, psi, chi = (np.full(case["m"], x) for x in v)
        if not case["quasi"]:
            psi, chi = 0.0 * psi, 0.0 * chi
    sizes = torch.tensor(np.diff(off), device=DEV)
    idx = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)
    a, b, c = (torch.tensor(v, **dev)[idx] for v in (tm1, t0, t1))
    first, last = torch.tensor(off[:-1], device=DEV), torch.tensor(off[1:] - 1, device=DEV)
    b[first] += torch.tensor(psi, **dev)
    b[last] += torch.tensor(chi, **dev)
    a[first], c[last] = 0.0, 0.0
    return a, b, c, idx, int(sizes.max())


def _sines(n):
    """The sine matrix with exact argument reduction, and (2/h sin)^2."""
    q = torch.arange(1, n + 1, dtype=torch.int64, device=DEV)
    r = (q[:, None] * q[None, :]) % (2 * (n + 1))
    S = torch.sin(math.pi * r.to(torch.float64) / (n + 1))
    lam = (2.0 * (n + 1) * torch.sin(math.pi * q.to(torch.float64) / (2 * (n + 1)))) ** 2
    return S, lam


def exact(case, seed):
    kind = case["kind"]
    F, W = _inputs(case, seed)
    if kind in ("poisson2d", "poisson3d"):
        # every direction diagonalised by its sine matrix
        dims = [case["nz"]] if kind == "poisson3d" else []
        dims += [case["ny"], case["nx"]]
        mats = [_sines(n) for n in dims]

        def transform(V):
            for d, (S, _) in enumerate(mats):
                V = torch.movedim(V, d, -1)
                V = torch.movedim((V.reshape(-1, S.shape[0]) @ S).reshape(V.shape), -1, d)
            return V.contiguous()

        V = transform(F)
        lam = 0.0
        for d, (_, l) in enumerate(mats):
            lam = lam + l.reshape([-1 if k == d else 1 for k in range(len(dims))])
        V /= lam
        for n in dims:
            V *= 2.0 / (n + 1)
        return transform(V)
    if kind == "strided":
        n, m, nb = case["n"], case["m"], case["nb"]
        tm1, t0, t1 = _strided_matrix(case, seed)
        b = torch.tensor(t0, dtype=torch.float64, device=DEV)[None, :, None]
        b = b.expand(nb, m, n).reshape(-1).contiguous()
        a, c = torch.full_like(b, tm1), torch.full_like(b, t1)
        a[::n], c[n - 1::n] = 0.0, 0.0
        f = F.transpose(1, 2).contiguous().reshape(-1)
        return _solve_flat(a, b, c, f, n).reshape(nb, m, n).transpose(1, 2).contiguous()
    a, b, c, idx, longest = _flat_rows(case, seed)
    dt = F.dtype
    X = _solve_flat(a, b, c, F.to(torch.float64).reshape(-1), longest)
    if W is None:
        return X.reshape(F.shape)
    # the transposed matrix: its lower entries are c moved down, its upper a moved up
    gF = _solve_flat(_shift(c, 1), b, _shift(a, -1), W.to(torch.float64).reshape(-1), longest)
    # the entry gradients against the forward solution; a and c are 0 where a
    # row has no such neighbour
    ga = torch.where(a == 0, 0.0, -gF * _shift(X, 1))
    gb = -gF * X
    gc = torch.where(c == 0, 0.0, -gF * _shift(X, -1))
    if kind == "general":
        g = torch.stack([v.reshape(case["m"], -1).sum(0) for v in (ga, gb, gc)])
        return X.reshape(F.shape), gF.reshape(F.shape), g
    cols = [ga, gb, gc]
    if case["quasi"]:   # the corners' terms, on the first and last rows
        cols += [torch.where(a == 0, gb, 0.0), torch.where(c == 0, gb, 0.0)]
    if kind == "varlen":
        sizes = torch.bincount(idx).tolist()
        g = torch.stack([torch.stack([p.sum() for p in torch.split(v, sizes)]) for v in cols], 1)
    else:
        g = torch.stack([v.sum() for v in cols])
    if kind == "autograd":
        g = g.cpu()
    return X.reshape(F.shape), gF.reshape(F.shape), g
