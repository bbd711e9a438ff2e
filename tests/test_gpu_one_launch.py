"""Solves that form their tiles' outside values in the final pass, and the
other one-launch and few-launch paths, on what their parity tests leave open:
the gradients by component, which route a solve takes (the launches of its
captured graph), right-hand sides with NaN and infinities, and graph replays.

Tolerances: X and gF those of the parity tests.  A gradient is a sum of
products of the device's own gF and X, formed in double in a tree of at most
64 additions: 64 u of the products' mass, component by component; a float
plan's corner terms come from corner unknowns before their rounding to float,
2^-24 of these terms' mass more."""
import numpy as np
import pytest

import oracle
from gpu_util import U64, to_dev, to_host, tol_f32, tol_f64
from test_gpu_halo import TILE, _row_err
from test_gpu_quasi import quasi_system
from test_gpu_short_routes import gradient_and_mass

pytestmark = pytest.mark.gpu


def _tdt():
    import paper_1002_2469_amd as tdt
    return tdt


def _launches(fn):
    from gpu_graph import captured, nodes
    return nodes(captured(fn))


@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("ratio,extra,one", [(3.0, 0, True), (3.0, 250, True), (3.0, 1, False),
                                             (1.1, 0, True), (1.1, 250, True),
                                             (1.012, 0, True), (1.012, 250, False)])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_gradients_and_route(dtype, quasi, ratio, extra, one, shape):
    """one: supports short enough for the last tile (none fits in 1 row, 320
    and more rows of ratio 1.012 not in 250)."""
    import torch
    n = 3 * TILE[shape] + extra
    rng = np.random.default_rng(extra + shape)
    a = c = -1.0
    b = 2.0 * ratio
    tol = tol_f32(a, b, c, n) if dtype == "f32" else tol_f64(a, b, c, n)
    q = dict(psi=0.7, chi=0.4) if quasi else {}
    N = n + 2 * quasi
    plan = _tdt().Plan(a, b, c, N, dtype, **q)
    plan.set_option("shape", shape)
    F, W = rng.standard_normal((2, 3, N))
    if dtype == "f32":
        F, W = (v.astype(np.float32).astype(np.float64) for v in (F, W))
    print(f"[case] one launch n={n} ratio={ratio} shape={shape} {dtype} quasi={quasi}", flush=True)
    Fd, Wd = to_dev(F, dtype), to_dev(W, dtype)
    Xd = plan.solve(Fd)
    gFd, gtd = plan.backward(Wd, Xd)
    X, gF, gt = to_host(Xd), to_host(gFd), to_host(gtd)
    assert _row_err(X, oracle.solve(F, a, b, c, **q)) <= tol
    gFr, _ = oracle.adjoint(W, X, a, b, c, corners=quasi, **q)
    assert _row_err(gF, gFr) <= tol
    ref, mass = gradient_and_mass(gF, X, quasi)
    bound = 64 * U64 * mass
    if dtype == "f32" and quasi:
        bound = bound + 2.0 ** -24 * sum(gradient_and_mass(gF[:, i], X[:, i], True)[1]
                                         for i in (slice(0, 2), slice(-2, None)))
    assert np.all(np.abs(gt - ref) <= bound), (gt, ref, bound)
    out = torch.empty_like(Fd)
    assert (_launches(lambda: plan.solve(Fd, out)) == 1) == one


@pytest.mark.parametrize("M,shape,one", [(64, 0, True), (75, 0, False), (32, 1, True),
                                         (40, 1, False), (64, 2, True), (85, 2, False)])
def test_float_route_by_tiles(M, shape, one):
    """Float series with 512 support rows: one launch while the tiles are about
    one round of resident workgroups."""
    import torch
    n, a, b, c = 65536, -1.0, 2.04, -1.0
    plan = _tdt().Plan(a, b, c, n, "f32")
    plan.set_option("shape", shape)
    assert sum(plan.green_support()["forward"]) == 512
    F = np.random.default_rng(M).standard_normal((M, n)).astype(np.float32).astype(np.float64)
    Fd = to_dev(F, "f32")
    out = torch.empty_like(Fd)
    print(f"[case] float route M={M} shape={shape}", flush=True)
    assert _row_err(to_host(plan.solve(Fd)), oracle.solve(F, a, b, c)) <= tol_f32(a, b, c, n)
    assert (_launches(lambda: plan.solve(Fd, out)) == 1) == one


BAD = {1: np.nan, 2: np.inf, 4: -np.inf}


@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_one_launch_series_do_not_meet(dtype, quasi, shape):
    """NaN and infinities, also next to the tiles' edges, leave the other
    right-hand sides exactly as without them and show in their own."""
    L = TILE[shape]
    n = 3 * L + 300
    rng = np.random.default_rng(shape)
    a, b, c, psi, chi = quasi_system(rng, 1.25)
    plan = _tdt().Plan(a, b, c, n, dtype, **(dict(psi=psi, chi=chi) if quasi else {}))
    plan.set_option("shape", shape)
    F = rng.standard_normal((6, n))
    print(f"[case] one launch isolation {dtype} quasi={quasi} shape={shape}", flush=True)
    X0 = to_host(plan.solve(to_dev(F, dtype)))
    for rows in ([0], [L - 1], [L + 1], [L // 2], [n - 1]):
        G = F.copy()
        for m, v in BAD.items():
            G[m, rows] = v
        X1 = to_host(plan.solve(to_dev(G, dtype)))
        good = [m for m in range(6) if m not in BAD]
        assert np.array_equal(X0[good], X1[good]), rows
        for m in BAD:
            assert not np.isfinite(X1[m, rows]).any(), (m, rows)


@pytest.mark.parametrize("M,nb,n", [(40, 2, 2000), (33, 1, 17 * 512 + 40)])
def test_strided_columns_do_not_meet(M, nb, n):
    """The same for the columns of tiled strided solves, their interface
    eliminated in the second pass (4 tiles) and in a launch of its own (18)."""
    rng = np.random.default_rng(M)
    t0 = rng.uniform(2.3, 4.0, M)
    plan = _tdt().StridedPlan(n, -1.0, t0, -1.0)
    F = rng.standard_normal((nb, n, M))
    print(f"[case] strided isolation M={M} n={n}", flush=True)

    def solve(v):
        return to_host(plan.solve(to_dev(v), M=M, ld=M, nb=nb, ldb=n * M))
    X0 = solve(F)
    bad = {0: np.nan, 5: np.inf, 16: -np.inf, M - 1: np.nan}
    good = [k for k in range(M) if k not in bad]
    for row in (0, 511, 513, 700, n - 1):
        G = F.copy()
        for k, v in bad.items():
            G[0, row, k] = v
        X1 = solve(G)
        assert np.array_equal(X0[:, :, good], X1[:, :, good]) and np.array_equal(X0[1:], X1[1:])
        assert not np.isfinite(X1[0, row, list(bad)]).any(), row


@pytest.mark.parametrize("dims", [(99, 40), (127, 40), (100, 40), (99, 1200), (520, 30),
                                  (17, 30, 20), (18, 16, 18), (63, 127, 20)])
def test_poisson_after_nan(dims):
    """A right-hand side with a NaN gives one, and leaves nothing behind for
    the handle's next solve (work arrays, padding of odd row lengths)."""
    tdt = _tdt()
    F = np.random.default_rng(3).standard_normal(dims[::-1])
    s = (tdt.Poisson2D(*dims, 0.02, 0.03) if len(dims) == 2 else
         tdt.Poisson3D(*dims, 0.02, 0.03, 0.04))
    print(f"[case] poisson after nan {dims}", flush=True)
    U0 = to_host(s.solve(to_dev(F)))
    G = F.copy()
    G.flat[F.size // 2] = np.nan
    assert np.isnan(to_host(s.solve(to_dev(G)))).any()
    assert np.array_equal(to_host(s.solve(to_dev(F))), U0)


def _plan_cases():
    tdt = _tdt()
    rng = np.random.default_rng(9)
    off = np.array([0, 700, 1724, 1800, 2500], dtype=np.int64)
    big = np.array([0, 20000, 36384, 60000], dtype=np.int64)
    q = dict(psi=0.4, chi=0.5)
    return {
        "halo": (tdt.Plan(-0.9, 2.5, -1.1, 30011), "f64", (5, 30011)),
        "halo quasi refine": (tdt.Plan(-0.9, 2.5, -1.1, 30011, "f32_refine", **q), "f64",
                              (5, 30011)),
        "short": (tdt.Plan(-0.9, 2.5, -1.1, 255), "f64", (3000, 255)),
        "short quasi refine": (tdt.Plan(-0.9, 2.5, -1.1, 255, "f32_refine", **q), "f64",
                               (3000, 255)),
        "short float": (tdt.Plan(-0.9, 2.5, -1.1, 255, "f32"), "f32", (3000, 255)),
        "short batch": (tdt.VarlenPlan(off, -0.9, rng.uniform(2.5, 4, 4), -1.1), "f64", (2500,)),
        "halo batch": (tdt.VarlenPlan(big, -0.9, rng.uniform(2.5, 4, 3), -1.1), "f64", (60000,)),
    }


@pytest.mark.parametrize("name", ["halo", "halo quasi refine", "short", "short quasi refine",
                                  "short float", "short batch", "halo batch"])
def test_plan_graph_replays(name):
    import torch
    from gpu_graph import captured, replays_agree
    plan, dt, shape = _plan_cases()[name]
    rng = np.random.default_rng(1)
    F, W = (to_dev(rng.standard_normal(shape), dt) for _ in range(2))
    print(f"[case] graph {name}", flush=True)
    X = plan.solve(F)
    gF, gt = plan.backward(W, X)
    out = [torch.empty_like(v) for v in (X, gF, gt)]

    def run():
        plan.solve(F, out[0])
        plan.backward(W, out[0], out[1], out[2])
    assert replays_agree(captured(run), out, [X, gF, gt])


@pytest.mark.parametrize("dims", [(99, 40), (100, 1200), (127, 1500), (30, 50), (17, 30, 20),
                                  (18, 16, 18), (127, 63, 20)])
def test_poisson_graph_replays(dims):
    import torch
    from gpu_graph import captured, replays_agree
    tdt = _tdt()
    F = to_dev(np.random.default_rng(3).standard_normal(dims[::-1]))
    s = (tdt.Poisson2D(*dims, 0.02, 0.03) if len(dims) == 2 else
         tdt.Poisson3D(*dims, 0.02, 0.03, 0.04))
    print(f"[case] graph poisson {dims}", flush=True)
    U = s.solve(F)
    out = torch.empty_like(U)
    assert replays_agree(captured(lambda: s.solve(F, out)), [out], [U])


@pytest.mark.parametrize("M,nb,n", [(40, 2, 2000), (33, 1, 17 * 512 + 40)])
def test_strided_graph_replays(M, nb, n):
    import torch
    from gpu_graph import captured, replays_agree
    rng = np.random.default_rng(M)
    plan = _tdt().StridedPlan(n, -1.0, rng.uniform(2.3, 4.0, M), -1.0)
    F = to_dev(rng.standard_normal((nb, n, M)))
    kw = dict(M=M, ld=M, nb=nb, ldb=n * M)
    print(f"[case] graph strided M={M} n={n}", flush=True)
    X = plan.solve(F, **kw)
    out = torch.empty_like(X)
    assert replays_agree(captured(lambda: plan.solve(F, out, **kw)), [out], [X])
