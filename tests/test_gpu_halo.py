"""GPU parity of solves whose final pass forms the values outside its tiles
itself (one launch), against the CPU oracle, through the C ABI: supports of one
run of 64 rows, of as many as are requested ahead (128 + 128), of more, and the
longest a tile takes; a whole and a ragged last tile, one just long enough for
the supports' entries and one too short for them (which takes the separate
passes); quasi-Toeplitz ends; series, batches, every work shape; forward and
adjoint; and a batch with one system that cannot, which must agree.

Inputs: right-hand sides scaled apart by many orders of magnitude, each checked
against its own norm; symmetric matrices of the stated dominance (and
unsymmetric ones in the batches).  Tolerances: the tiers of the other tests."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host, tol_f32, tol_f64
from test_gpu_quasi import quasi_system

pytestmark = pytest.mark.gpu
TILE = {0: 8192, 1: 4096, 2: 4096}


def _tdt():
    import paper_1002_2469_amd as tdt
    return tdt


def _row_err(x, ref):
    return float((np.abs(x - ref).max(-1) / np.abs(ref).max(-1)).max())


@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("ratio", [3.0, 1.1, 1.05, 1.012])
@pytest.mark.parametrize("extra", [0, 1, 250, 700, 2000, 4095])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_halo_series(dtype, extra, ratio, shape):
    tdt = _tdt()
    n = 3 * TILE[shape] + extra
    rng = np.random.default_rng(extra + shape)
    a = c = -1.0
    b = 2.0 * ratio
    tol = tol_f32(a, b, c, n) if dtype == "f32" else tol_f64(a, b, c, n)
    for quasi in (False, True):
        q = dict(psi=0.7, chi=0.4) if quasi else {}
        plan = tdt.Plan(a, b, c, n + 2 * quasi, dtype, **q)
        plan.set_option("shape", shape)
        F = rng.standard_normal((3, n + 2 * quasi)) * 10.0 ** rng.integers(-9, 9, size=(3, 1))
        W = rng.standard_normal(F.shape)
        if dtype == "f32":
            F, W = (v.astype(np.float32).astype(np.float64) for v in (F, W))
        print(f"[case] halo n={n} ratio={ratio} shape={shape} {dtype} quasi={quasi} "
              f"supports={plan.green_support()}", flush=True)
        X = to_host(plan.solve(to_dev(F, dtype)))
        assert _row_err(X, oracle.solve(F, a, b, c, **q)) <= tol
        gF, gt = plan.backward(to_dev(W, dtype), to_dev(X, dtype))
        gFr, gtr = oracle.adjoint(W, X, a, b, c, corners=quasi, **q)
        assert _row_err(to_host(gF), gFr) <= tol
        mass = (np.abs(gFr).sum(1) * np.abs(X).max(1)).sum()
        assert np.abs(to_host(gt) - gtr).max() <= 10 * tol * mass


@pytest.mark.parametrize("weak", [False, True])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_halo_varlen(dtype, quasi, weak):
    """weak: one system whose last tile is too short for the entries, so that
    the whole batch takes the separate passes."""
    tdt = _tdt()
    rng = np.random.default_rng(6)
    sizes = [8192, 9000, 16384, 30000, 65536, 8193 + 4000, 5000, 100000] + [8192 + 9] * weak
    sizes = np.array(sizes) + 2 * quasi
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    t = np.array([quasi_system(rng, 1.25) for _ in sizes]).T
    q = dict(psi=t[3], chi=t[4]) if quasi else {}
    scale = np.repeat(10.0 ** rng.integers(-9, 9, size=len(sizes)), sizes)
    F, W = rng.standard_normal(off[-1]) * scale, rng.standard_normal(off[-1])
    if dtype == "f32":
        F, W = (v.astype(np.float32).astype(np.float64) for v in (F, W))
    tol = 2e-5 if dtype == "f32" else 1e-12
    plan = tdt.VarlenPlan(off, t[0], t[1], t[2], dtype, **q)
    for whole in (8, 0):
        print(f"[case] halo varlen {dtype} quasi={quasi} weak={weak} whole={whole}", flush=True)
        plan.set_option("whole_max_tiles", whole)
        X = to_host(plan.solve(to_dev(F, dtype)))
        gF, gt = (to_host(v) for v in plan.backward(to_dev(W, dtype), to_dev(X, dtype)))
        ref = oracle.solve_varlen(F, off, t[0], t[1], t[2], **q)
        gFr, gtr = oracle.adjoint_varlen(W, X, off, t[0], t[1], t[2], corners=quasi, **q)
        for s in range(len(sizes)):
            i = slice(off[s], off[s + 1])
            assert _row_err(X[None, i], ref[None, i]) <= tol, (s, sizes[s])
            assert _row_err(gF[None, i], gFr[None, i]) <= tol, (s, sizes[s])
            mass = np.abs(gFr[i]).sum() * np.abs(X[i]).max()
            assert np.abs(gt[s] - gtr[s]).max() <= 10 * tol * mass, (s, sizes[s])
