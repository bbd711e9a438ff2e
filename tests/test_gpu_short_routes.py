"""GPU parity of short series on both sides of the lines between the tile
kernels, one system per narrow workgroup and several per workgroup: numbers of
systems that the device holds at once in the narrowest workgroups, and one
more; refined plans at a few systems, around three quarters of the device, and
above; forward and adjoint, the gradients by component.

Tolerances: X and gF those of the other short-system tests.  A gradient is a
sum of products of the device's own gF and X, formed in double in a tree of at
most 64 additions: 64 u of the products' mass, component by component."""
import numpy as np
import pytest

import oracle
from gpu_util import U64, to_dev, to_host
from test_gpu_quasi import quasi_system
from test_gpu_short import TOL, _row_err

pytestmark = pytest.mark.gpu


def gradient_and_mass(gF, X, quasi):
    """The t-gradients from gF and X [M][n], and the sums of the products'
    magnitudes."""
    gF, X = (np.asarray(v, np.longdouble) for v in (gF, X))
    terms = [gF[:, 1:] * X[:, :-1], gF * X, gF[:, :-1] * X[:, 1:]]
    if quasi:
        terms += [gF[:, :1] * X[:, :1], gF[:, -1:] * X[:, -1:]]
    return (np.array([-t.sum() for t in terms], np.float64),
            np.array([np.abs(t).sum() for t in terms], np.float64))


# 1500 rows: 128 lanes, 2048 of which the device holds; 4096: 256 lanes, 1024;
# refined plans: 384 workgroups of 512 lanes are three quarters of it
@pytest.mark.parametrize("n,Ms", [(300, (1, 383, 385)), (1500, (3, 383, 385, 2048, 2049)),
                                  (2100, (3, 385, 1024, 1025)), (4094, (5, 384, 1025))])
@pytest.mark.parametrize("quasi", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32_refine", "f32"])
def test_short_routes(n, Ms, dtype, quasi):
    import paper_1002_2469_amd as tdt
    rng = np.random.default_rng(n)
    a, b, c, psi, chi = quasi_system(rng, 1.25)
    q = dict(psi=psi, chi=chi) if quasi else {}
    plan = tdt.Plan(a, b, c, n, dtype, **q)
    for M in Ms:
        print(f"[case] short routes n={n} M={M} {dtype} quasi={quasi}", flush=True)
        F = rng.standard_normal((M, n)) * 10.0 ** rng.integers(-9, 9, size=(M, 1))
        W = rng.standard_normal((M, n))
        if dtype == "f32":
            F, W = (v.astype(np.float32).astype(np.float64) for v in (F, W))
        X = plan.solve(to_dev(F, dtype))
        gF, gt = plan.backward(to_dev(W, dtype), X)
        X, gF, gt = to_host(X), to_host(gF), to_host(gt)
        assert _row_err(X, oracle.solve(F, a, b, c, **q)) <= TOL[dtype]
        gFr, _ = oracle.adjoint(W, X, a, b, c, corners=quasi, **q)
        assert _row_err(gF, gFr) <= TOL[dtype]
        ref, mass = gradient_and_mass(gF, X, quasi)
        tol = 64 * U64 * mass
        if dtype == "f32" and quasi:
            # the corner rows' terms come from their unrounded unknowns
            _, corner = gradient_and_mass(gF[:, :2], X[:, :2], True)
            _, last = gradient_and_mass(gF[:, -2:], X[:, -2:], True)
            tol = tol + 2.0 ** -24 * (corner + last)
        assert np.all(np.abs(gt - ref) <= tol), (gt, ref, tol)
