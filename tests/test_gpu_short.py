"""GPU parity of the short-system path (several systems per workgroup, a few
blocks of 16 rows each) against the CPU oracle, through the C ABI: sizes at
the edges of blocks, wavefronts and workgroup widths, right-hand side counts
that leave the last run partial, quasi-Toeplitz ends, varlen batches, the
adjoint, and that a system's values never reach its neighbours.

Inputs: dominance ratio in [1.25, 3]; right-hand sides whose scales differ by
many orders of magnitude between the systems of one workgroup, each checked
against its own norm.  Tolerances: the tiers of the other parity tests."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host
from paper_1002_2469_amd import workloads as W
from test_gpu_quasi import quasi_system

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32_refine": 1e-12, "f32": 2e-5}
# one row; a block less, equal and more; 16 blocks (a row of lanes); the ends
# of a wavefront's (1024) and of the wider workgroups' (2048, 4096) ranges
SIZES = [1, 2, 15, 16, 17, 33, 255, 256, 257, 513, 1008, 1023, 1024, 1025, 1365, 2047, 2049,
         4096]


def _tdt():
    import paper_1002_2469_amd as tdt
    return tdt


def _rhs(rng, M, n, dtype):
    scale = 10.0 ** rng.integers(-12, 12, size=(M, 1))
    F = rng.standard_normal((M, n)) * scale
    return F.astype(np.float32).astype(np.float64) if dtype == "f32" else F


def _row_err(x, ref):
    return float((np.abs(x - ref).max(-1) / np.abs(ref).max(-1)).max())


@pytest.mark.parametrize("shape", [0, 2])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
@pytest.mark.parametrize("n", SIZES)
def test_short_series(n, dtype, quasi, shape):
    tdt = _tdt()
    n += 2 if quasi else 0
    rng = np.random.default_rng(17 * n + shape)
    a, b, c, psi, chi = quasi_system(rng, 1.25)
    q = dict(psi=psi, chi=chi) if quasi else {}
    plan = tdt.Plan(a, b, c, n, dtype, **q)
    plan.set_option("shape", shape)
    for M in (1, 2, 37):
        print(f"[case] short n={n} M={M} {dtype} quasi={quasi} shape={shape}", flush=True)
        F, Wt = _rhs(rng, M, n, dtype), _rhs(rng, M, n, dtype)
        X = to_host(plan.solve(to_dev(F, dtype)))
        assert _row_err(X, oracle.solve(F, a, b, c, **q)) <= TOL[dtype]
        gF, gt = plan.backward(to_dev(Wt, dtype), to_dev(X, dtype))
        gFr, gtr = oracle.adjoint(Wt, X, a, b, c, corners=quasi, **q)
        assert _row_err(to_host(gF), gFr) <= TOL[dtype]
        # sums of products gF_i x_j: against a bound of the products' mass
        mass = (np.abs(gFr).sum(1) * np.abs(X).max(1)).sum()
        assert np.abs(to_host(gt) - gtr).max() <= 10 * TOL[dtype] * mass


@pytest.mark.parametrize("long", [False, True])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_short_varlen(dtype, quasi, long):
    """A batch of systems up to 1024 rows (a wavefront each), and many of them
    next to longer ones on the other paths; forward and adjoint."""
    tdt = _tdt()
    rng = np.random.default_rng(3)
    sizes = [1, 16, 17, 1024, 255, 512, 2, 1023, 1008, 33]
    if long:
        sizes += list(rng.integers(1, 300, 1400)) + [9000, 1025, 30000, 8192, 1026]
    sizes = np.array(sizes)
    if quasi:
        sizes = np.maximum(sizes, 3)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    t = np.array([quasi_system(rng, 1.25) for _ in sizes]).T
    q = dict(psi=t[3], chi=t[4]) if quasi else {}
    scale = np.repeat(10.0 ** rng.integers(-12, 12, size=len(sizes)), sizes)
    F, Wt = rng.standard_normal(off[-1]) * scale, rng.standard_normal(off[-1]) * scale
    if dtype == "f32":
        F, Wt = (v.astype(np.float32).astype(np.float64) for v in (F, Wt))
    print(f"[case] short varlen {dtype} quasi={quasi} long={long}", flush=True)
    plan = tdt.VarlenPlan(off, t[0], t[1], t[2], dtype, **q)
    X = to_host(plan.solve(to_dev(F, dtype)))
    gF, gt = (to_host(v) for v in plan.backward(to_dev(Wt, dtype), to_dev(X, dtype)))
    ref = oracle.solve_varlen(F, off, t[0], t[1], t[2], **q)
    gFr, gtr = oracle.adjoint_varlen(Wt, X, off, t[0], t[1], t[2], corners=quasi, **q)
    for s in range(len(sizes)):
        i = slice(off[s], off[s + 1])
        assert _row_err(X[None, i], ref[None, i]) <= TOL[dtype], (s, sizes[s])
        assert _row_err(gF[None, i], gFr[None, i]) <= TOL[dtype], (s, sizes[s])
        mass = np.abs(gFr[i]).sum() * np.abs(X[i]).max()
        assert np.abs(gt[s] - gtr[s]).max() <= 10 * TOL[dtype] * mass, (s, sizes[s])


@pytest.mark.parametrize("n", [7, 100, 255, 600, 1400])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_short_systems_do_not_meet(dtype, quasi, n):
    """NaN, infinities and the largest values in some right-hand sides leave
    every other one exactly as without them."""
    tdt = _tdt()
    rng = np.random.default_rng(n)
    a, b, c, psi, chi = quasi_system(rng, 1.25)
    plan = tdt.Plan(a, b, c, n, dtype, **(dict(psi=psi, chi=chi) if quasi else {}))
    F = rng.standard_normal((23, n))
    print(f"[case] short isolation n={n} {dtype} quasi={quasi}", flush=True)
    X0 = to_host(plan.solve(to_dev(F, dtype)))
    bad = {1: np.nan, 4: np.inf, 9: -np.inf, 15: np.finfo(np.float32).max, 22: np.nan}
    for m, v in bad.items():
        F[m, [0, n // 2, n - 1]] = v
    X1 = to_host(plan.solve(to_dev(F, dtype)))
    good = [m for m in range(23) if m not in bad]
    assert np.array_equal(X0[good], X1[good])
    assert np.isnan(X1[1]).any() and np.isnan(X1[22]).any()


def test_short_workgroup_cap_keeps_bits():
    """Persistent workgroups (a cap per compute unit) loop over the runs and
    change no bit."""
    tdt = _tdt()
    rng = np.random.default_rng(8)
    n, M = 300, 40000
    plan = tdt.Plan(-0.9, 2.6, -1.1, n)
    F = to_dev(rng.standard_normal((M, n)))
    print("[case] short workgroup cap", flush=True)
    X = to_host(plan.solve(F))
    plan.set_option("wg_per_cu", 1)
    assert np.array_equal(to_host(plan.solve(F)), X)
