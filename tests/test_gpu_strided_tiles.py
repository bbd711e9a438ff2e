"""GPU parity of tiled strided solves whose first pass reads only the stretch
of the tiles' Green rows that carries their mass, next to groups of classes
whose tiles are swept, and of the interface elimination inside the second
pass, against the CPU oracle, through the C ABI.

Inputs: groups of 16 classes that are strongly dominant (short supports), just
inside and outside the longest support taken, weakly dominant (swept), of
either sign and with t_-1 t_1 < 0; orders whose last tile is 1 row, shorter
than the supports, and whole; up to and past the number of tiles eliminated
inside the second pass.  Tolerance: 1e-12 or 4 u cond(T) per system."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host, tol_f64

pytestmark = pytest.mark.gpu


def _tdt():
    import paper_1002_2469_amd as tdt
    return tdt


def classes(rng, P):
    """One kind per group of 16."""
    a, b, c = (np.empty(P) for _ in range(3))
    for k in range(P):
        kind = (k // 16) % 6
        a[k], c[k] = rng.uniform(0.4, 1.0, 2)
        ratio = {0: rng.uniform(1.5, 3.0), 1: 1.0005, 2: 1.06, 3: 1.03, 4: rng.uniform(1.2, 2.0),
                 5: rng.uniform(1.1, 1.5)}[kind]
        if kind in (1, 2, 3):
            c[k] = a[k]
        if kind == 4:
            a[k] = -a[k]
        if kind == 5:
            a[k], c[k] = -a[k], -c[k]
        b[k] = ratio * (abs(a[k]) + abs(c[k])) * (1 if k % 2 else -1)
    if P > 20:
        c[20] = 0.0     # a bidiagonal class in a swept group
    return a, b, c


@pytest.mark.parametrize("n", [1025, 1034, 1100, 1536, 2000, 16 * 512, 16 * 512 + 200, 9001])
@pytest.mark.parametrize("M,nb", [(1, 1), (33, 2), (200, 1), (96, 5)])
def test_strided_supports(n, M, nb):
    tdt = _tdt()
    rng = np.random.default_rng(n + M)
    a, b, c = classes(rng, M + 3)
    F = rng.standard_normal((nb, n, M)) * 10.0 ** rng.integers(-8, 8, size=(nb, 1, M))
    print(f"[case] strided supports n={n} M={M} nb={nb}", flush=True)
    plan = tdt.StridedPlan(n, a, b, c)
    Fd = to_dev(F)
    X = to_host(plan.solve(Fd, M=M, ld=M, nb=nb, ldb=n * M))
    plan.solve(Fd, Fd, M=M, ld=M, nb=nb, ldb=n * M)   # in place
    assert np.array_equal(to_host(Fd), X)
    for k in range(M):
        ref = oracle.solve(np.ascontiguousarray(F[:, :, k]), a[k], b[k], c[k])
        err = np.abs(X[:, :, k] - ref).max(1) / np.abs(ref).max(1)
        assert err.max() <= tol_f64(a[k], b[k], c[k], n), (k, err.max())
