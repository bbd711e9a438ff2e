"""GPU parity of general tridiagonal plans whose last tile is ragged and whose
first pass reads the supports of the tiles' own Green rows, and of the entry
gradients summed in slices, against the CPU oracle, through the C ABI: last
tiles of 1 row, shorter and longer than the supports; row counts below,
between and above the slices' thresholds; M of 1, few and many.

Inputs: dominance ratio in [1.2, 3]; the rows past every right-hand side are
those of the next one, with values that would show."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host
from test_gpu_general import L, TOL, _f32_round, random_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M", [(L + 1, 7), (2 * L + 30, 5), (3 * L - 1, 1), (2 * L + 1000, 40),
                                 (3, 5000), (17, 3), (1000, 700), (20000, 9), (70000, 4),
                                 (300001, 2)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_general_ragged(n, M, dtype):
    import paper_1002_2469_amd as tdt
    rng = np.random.default_rng(n + M)
    a, b, c = random_rows(rng, n, 1.25, 3.0)
    F = _f32_round(rng.standard_normal((M, n)) * 1e3 ** rng.integers(-1, 2, size=(M, 1)), dtype)
    G = _f32_round(rng.standard_normal((M, n)), dtype)
    print(f"[case] general ragged n={n} M={M} {dtype}", flush=True)
    plan = tdt.GeneralPlan(a, b, c, dtype)
    Xd = plan.solve(to_dev(F, dtype))
    X = to_host(Xd)
    assert oracle.rel_err_rows(X, oracle.solve_general(F, a, b, c)).max() <= TOL[dtype]
    gF, g = plan.backward(to_dev(G, dtype), Xd)
    gFr, ref = oracle.adjoint_general(G, X, a, b, c)
    assert oracle.rel_err_rows(to_host(gF), gFr).max() <= TOL[dtype]
    ref = np.stack(ref)
    assert np.max(np.abs(to_host(g) - ref)) <= 10 * TOL[dtype] * np.max(np.abs(ref))
