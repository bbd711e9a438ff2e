"""The corner unknowns of refined quasi-Toeplitz systems of one tile (forward
and adjoint, series and batches, the widths of the short path) against a long
double elimination: their rows are eliminated in double, so their error is
that of a double solve, not of the refinement's stopping test.

Tolerance: 16 u of the largest unknown (u = 2^-53).  The elimination of a
tridiagonal matrix that is dominant by a ratio r without pivoting is off by at
most about 3 u |T^-1||T||x|, the row sums of |T^-1||T| are at most (1 + 1/r) /
(1 - 1/r) = 3 at r = 2, and the rounded constants of the chain add the same
order once more; the ratios here are 2 and 3."""
import numpy as np
import pytest

from gpu_util import U64, to_dev, to_host

pytestmark = pytest.mark.gpu


def _exact(F, a, b, c, psi, chi):
    """Thomas in long double, F [M][N]."""
    ld = np.longdouble
    F = F.astype(ld)
    a, b, c, psi, chi = (ld(v) for v in (a, b, c, psi, chi))
    M, N = F.shape
    cp, x = np.zeros(N, ld), np.zeros((M, N), ld)
    cp[0], x[:, 0] = c / (b + psi), F[:, 0] / (b + psi)
    for i in range(1, N):
        den = b + (chi if i == N - 1 else ld(0)) - a * cp[i - 1]
        cp[i], x[:, i] = c / den, (F[:, i] - a * x[:, i - 1]) / den
    for i in range(N - 2, -1, -1):
        x[:, i] -= cp[i] * x[:, i + 1]
    return x


def _check(X, ref, what):
    err = np.abs(X[:, [0, -1]] - ref[:, [0, -1]]).max(1) / np.abs(ref).max(1)
    assert err.max() <= 16 * U64, (what, float(err.max()))


@pytest.mark.parametrize("ratio", [2.0, 3.0])
@pytest.mark.parametrize("shape", [0, 2])
@pytest.mark.parametrize("n", [3, 17, 18, 35, 255, 1026, 2000, 4098, 8194])
def test_refined_corner_rows_series(n, shape, ratio):
    import paper_1002_2469_amd as tdt
    rng = np.random.default_rng(n)
    a, c, psi, chi = -0.93, -1.12, 0.41, 0.52
    b = ratio * (abs(a) + abs(c))
    plan = tdt.Plan(a, b, c, n, "f32_refine", psi=psi, chi=chi)
    plan.set_option("shape", shape)
    F, W = rng.standard_normal((2, 37, n))
    print(f"[case] corner rows n={n} shape={shape} ratio={ratio}", flush=True)
    X = plan.solve(to_dev(F))
    gF, _ = plan.backward(to_dev(W), X)
    _check(to_host(X), _exact(F, a, b, c, psi, chi), "X")
    _check(to_host(gF), _exact(W, c, b, a, psi, chi), "gF")


def test_refined_corner_rows_batch():
    import paper_1002_2469_amd as tdt
    rng = np.random.default_rng(5)
    sizes = np.array([3, 18, 19, 34, 100, 255, 513, 1000, 1023, 1024])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    a, c, psi, chi = rng.uniform(-1.0, -0.5, (4, len(sizes)))
    b = 3.0 * (abs(a) + abs(c))
    psi, chi = -0.4 * psi, -0.4 * chi
    F, W = rng.standard_normal((2, off[-1]))
    print("[case] corner rows batch", flush=True)
    plan = tdt.VarlenPlan(off, a, b, c, "f32_refine", psi=psi, chi=chi)
    X = plan.solve(to_dev(F))
    gF, _ = plan.backward(to_dev(W), X)
    X, gF = to_host(X), to_host(gF)
    for s in range(len(sizes)):
        i = slice(off[s], off[s + 1])
        _check(X[None, i], _exact(F[None, i], a[s], b[s], c[s], psi[s], chi[s]), (s, "X"))
        _check(gF[None, i], _exact(W[None, i], c[s], b[s], a[s], psi[s], chi[s]), (s, "gF"))
