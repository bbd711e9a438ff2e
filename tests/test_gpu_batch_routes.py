"""GPU parity of varlen batches on both sides of the lines between the
whole-system kernel and the paths that replace it: refined batches of short
systems (256 workgroups of 512 lanes, 768 of 256 are half and three quarters of
the device), float batches of one-tile quasi-Toeplitz systems (one round of
workgroups); forward and adjoint, the gradients by component.

Tolerances: X and gF those of the other short-system tests.  A gradient is a
sum of products of the device's own gF and X, formed in double in a tree of at
most 64 additions: 64 u of the products' mass, component by component; a float
plan's corner terms come from corner unknowns before their rounding to float,
2^-24 of these terms' mass more."""
import numpy as np
import pytest

import oracle
from gpu_util import U64, to_dev, to_host
from test_gpu_quasi import quasi_system
from test_gpu_short import TOL, _row_err
from test_gpu_short_routes import gradient_and_mass

pytestmark = pytest.mark.gpu


def _check_batch(sizes, dtype, quasi, shape, ratio=1.25):
    import paper_1002_2469_amd as tdt
    rng = np.random.default_rng(len(sizes))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    t = np.array([quasi_system(rng, ratio) for _ in sizes]).T
    q = dict(psi=t[3], chi=t[4]) if quasi else {}
    F, W = rng.standard_normal((2, off[-1]))
    if dtype == "f32":
        F, W = (v.astype(np.float32).astype(np.float64) for v in (F, W))
    plan = tdt.VarlenPlan(off, t[0], t[1], t[2], dtype, **q)
    plan.set_option("shape", shape)
    X = plan.solve(to_dev(F, dtype))
    gF, gt = plan.backward(to_dev(W, dtype), X)
    X, gF, gt = to_host(X), to_host(gF), to_host(gt)
    ref = oracle.solve_varlen(F, off, t[0], t[1], t[2], **q)
    gFr, _ = oracle.adjoint_varlen(W, X, off, t[0], t[1], t[2], corners=quasi, **q)
    for s in range(len(sizes)):
        i = slice(off[s], off[s + 1])
        assert _row_err(X[None, i], ref[None, i]) <= TOL[dtype], s
        assert _row_err(gF[None, i], gFr[None, i]) <= TOL[dtype], s
        g, mass = gradient_and_mass(gF[None, i], X[None, i], quasi)
        bound = 64 * U64 * mass
        if dtype == "f32" and quasi:
            bound = bound + 2.0 ** -24 * sum(
                gradient_and_mass(gF[None, i][:, e], X[None, i][:, e], True)[1]
                for e in (slice(0, 2), slice(-2, None)))
        assert np.all(np.abs(gt[s] - g) <= bound), (s, gt[s], g, bound)


@pytest.mark.parametrize("shape,S", [(0, 1), (0, 256), (0, 257), (2, 768), (2, 769)])
@pytest.mark.parametrize("quasi", [False, True])
def test_refined_short_batches(quasi, shape, S):
    print(f"[case] short batch S={S} shape={shape} quasi={quasi}", flush=True)
    sizes = np.random.default_rng(S).integers(3, 1025, S)
    sizes[0] = 1024
    _check_batch(sizes, "f32_refine", quasi, shape)


@pytest.mark.parametrize("shape,S", [(0, 512), (0, 513), (2, 1024), (2, 1025)])
@pytest.mark.parametrize("ratio", [1.25, 1.9])
def test_float_one_tile_batches(ratio, shape, S):
    """Quasi-Toeplitz systems of one tile, longer than the short ones: up to a
    round of workgroups (512 of 512 lanes, 1024 of 256) forward by the tile
    kernel, above by the whole-system kernel; the adjoint by the tile kernel."""
    print(f"[case] float one-tile batch S={S} shape={shape} ratio={ratio}", flush=True)
    sizes = np.random.default_rng(S).integers(1025, (8192 if shape == 0 else 4096) + 1, S)
    sizes[0] = 8194 if shape == 0 else 4098
    _check_batch(sizes, "f32", True, shape, ratio)
