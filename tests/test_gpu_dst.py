"""GPU parity of the mixed-radix sine transforms (rows and columns) through the
Poisson solves: every radix, the edges of the thread counts (n just above and
at 8 times a power of two), odd and even row and column counts, against the
CPU oracle; and the ADI iterate in closed form against the oracle's literal
iteration at loose and tight eps.

Inputs and tolerances: those of the other Poisson tests."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host
from oracle import poisson2d as P2
from oracle import poisson3d as P3
from test_gpu_poisson import tol as tol2
from test_gpu_poisson3d import _check_elementwise, _kappa, _tol

pytestmark = pytest.mark.gpu

# n = nx + 1: the radices alone and in powers, products of all of them, and
# the thread counts' edges (64 | 65, 128 | 130, 512 | 520, 1024 | 1040, ...)
NS = [2, 3, 4, 5, 6, 7, 11, 13, 9, 25, 49, 121, 169, 27, 60, 64, 65, 66, 130, 182, 243, 260,
      500, 520, 625, 1000, 1040, 1155, 2187, 2310, 4095, 5005, 6561]


def _tdt():
    import paper_1002_2469_amd as tdt
    return tdt


@pytest.mark.parametrize("n", NS)
@pytest.mark.parametrize("dtype", ["f64", "f32_refine"])
def test_dst_rows(n, dtype):
    """f64 takes the in-place line solves from 64 columns on, the transposes
    below and in f32_refine."""
    tdt = _tdt()
    nx = n - 1
    rng = np.random.default_rng(n)
    hx, hy = rng.uniform(0.002, 0.2, 2)
    for ny in (1, 2, 19):
        print(f"[case] dst rows n={n} ny={ny} {dtype}", flush=True)
        F = rng.standard_normal((ny, nx))
        U = to_host(tdt.Poisson2D(nx, ny, hx, hy, dtype).solve(to_dev(F)))
        err = oracle.rel_err(U, P2.solve(F, hx, hy))
        assert err <= tol2(nx, ny, hx, hy), (n, ny, err)


def test_dst_rows_line_plan():
    """Asking for the line plan of an in-place handle moves it to a varlen
    plan that takes options; solves before and after agree."""
    tdt = _tdt()
    rng = np.random.default_rng(4)
    nx, ny, hx, hy = 99, 20000, 0.01, 0.004
    F = rng.standard_normal((ny, nx))
    print("[case] dst line plan", flush=True)
    s = tdt.Poisson2D(nx, ny, hx, hy)
    ref = P2.solve(F, hx, hy)
    assert oracle.rel_err(to_host(s.solve(to_dev(F))), ref) <= tol2(nx, ny, hx, hy)
    s.set_line_option("whole_max_tiles", 0)
    assert oracle.rel_err(to_host(s.solve(to_dev(F))), ref) <= tol2(nx, ny, hx, hy)
    s.line_profile(True)
    s.solve(to_dev(F))
    assert s.line_profile_read()["solves"] == 1


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 6), (15, 11, 12), (16 - 1, 64, 65), (17, 7, 3),
                                  (20, 1, 1023), (33, 129, 25), (62, 24, 48), (127, 12, 519)])
@pytest.mark.parametrize("eps", [0.3, 1e-4, 1e-13])
def test_closed_iterate(dims, eps):
    """nx = 17, 62 keep one more entry after an odd or even last column."""
    tdt = _tdt()
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 100 + ny + nz)
    hx, hy, hz = rng.uniform(0.02, 0.1, 3)
    F = rng.standard_normal((nz, ny, nx))
    print(f"[case] closed iterate {dims} eps={eps}", flush=True)
    s = tdt.Poisson3D(nx, ny, nz, hx, hy, hz, eps)
    U = to_host(s.solve(to_dev(F)))
    counts, _ = s.schedule()
    ref = P3.solve(F, hx, hy, hz, eps=eps)
    _check_elementwise(U, ref, _tol(max(counts), _kappa(nx, ny, nz, hx, hy, hz)),
                       f"{dims} eps={eps}")
    assert np.array_equal(U, to_host(s.solve(to_dev(F))))


@pytest.mark.parametrize("dims", [(1, 63, 63), (5, 127, 63), (18, 63, 127), (33, 255, 127),
                                  (3, 127, 255), (2, 511, 255), (17, 255, 511), (1, 1023, 511),
                                  (16, 63, 1023)])
def test_closed_iterate_powers_of_two(dims):
    """Interval counts 8 T of the column transforms' thread counts: 64 (two
    radix-8 passes), 128 and 256 (a last pass of radix 2 and 4), 512, and 1024
    (two wavefronts per pair), along y and along z; columns short of a
    workgroup's sixteen and one more."""
    tdt = _tdt()
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 100 + ny + nz)
    hx, hy, hz = rng.uniform(0.02, 0.1, 3)
    F = rng.standard_normal((nz, ny, nx))
    print(f"[case] closed iterate {dims}", flush=True)
    s = tdt.Poisson3D(nx, ny, nz, hx, hy, hz, 1e-4)
    U = to_host(s.solve(to_dev(F)))
    counts, _ = s.schedule()
    ref = P3.solve(F, hx, hy, hz, eps=1e-4)
    _check_elementwise(U, ref, _tol(max(counts), _kappa(nx, ny, nz, hx, hy, hz)), f"{dims}")
    assert np.array_equal(U, to_host(s.solve(to_dev(F))))


@pytest.mark.parametrize("n,ny", [(60, 24603), (120, 12303), (250, 6202), (500, 3101), (1000, 1602),
                                  (2000, 801), (4095, 402)])
def test_dst_rows_many(n, ny):
    """Enough rows for the fewest threads per pair (few rows take two or four
    times as many: test_dst_rows)."""
    tdt = _tdt()
    rng = np.random.default_rng(n)
    hx, hy = rng.uniform(0.002, 0.2, 2)
    print(f"[case] dst rows n={n} ny={ny}", flush=True)
    F = rng.standard_normal((ny, n - 1))
    U = to_host(tdt.Poisson2D(n - 1, ny, hx, hy).solve(to_dev(F)))
    assert oracle.rel_err(U, P2.solve(F, hx, hy)) <= tol2(n - 1, ny, hx, hy)


@pytest.mark.parametrize("n", [17, 19, 51, 97, 127, 129, 131, 241, 254, 257, 262, 318, 323, 383, 502, 509, 521])
def test_dst_dense_rows(n):
    """Interval counts with a prime factor above 13: the matrix form up to 512
    (the edges of its LDS sizes: 127 | 129, 254 | 257, 318 | 323; odd and even),
    few rows (16 per workgroup) and many (32), ragged; 521: hipFFT."""
    tdt = _tdt()
    rng = np.random.default_rng(n)
    hx, hy = rng.uniform(0.002, 0.2, 2)
    for ny in (1, 37, 16389 if n <= 129 else 450):
        print(f"[case] dense rows n={n} ny={ny}", flush=True)
        F = rng.standard_normal((ny, n - 1))
        U = to_host(tdt.Poisson2D(n - 1, ny, hx, hy).solve(to_dev(F)))
        err = oracle.rel_err(U, P2.solve(F, hx, hy))
        assert err <= tol2(n - 1, ny, hx, hy), (n, ny, err)


@pytest.mark.parametrize("dims", [(1, 16, 18), (15, 50, 16), (33, 18, 60), (16, 127, 130),
                                  (50, 128, 33), (17, 256, 50), (3, 50, 261), (5, 382, 22),
                                  (2, 63, 508), (40, 508, 15), (33, 600, 37), (3, 16, 521),
                                  (400, 16, 82), (400, 82, 16), (64, 259, 130), (64, 259, 282),
                                  (64, 282, 259)])
@pytest.mark.parametrize("eps", [0.3, 1e-13])
def test_dense_iterate(dims, eps):
    """The matrix form along y, along z with the factors, or both, next to the
    FFT form; 16 and 32 columns per workgroup, ragged; (3, 16, 521) iterates."""
    tdt = _tdt()
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 100 + ny + nz)
    hx, hy, hz = rng.uniform(0.02, 0.1, 3)
    F = rng.standard_normal((nz, ny, nx))
    print(f"[case] dense iterate {dims} eps={eps}", flush=True)
    s = tdt.Poisson3D(nx, ny, nz, hx, hy, hz, eps)
    U = to_host(s.solve(to_dev(F)))
    counts, _ = s.schedule()
    ref = P3.solve(F, hx, hy, hz, eps=eps)
    _check_elementwise(U, ref, _tol(max(counts), _kappa(nx, ny, nz, hx, hy, hz)),
                       f"{dims} eps={eps}")
    assert np.array_equal(U, to_host(s.solve(to_dev(F))))


@pytest.mark.parametrize("dims", [(17, 190000, 1), (18, 180000, 1)])
def test_padded_rows_out_of_reach(dims):
    """Padded rows would pass the line solves' 31-bit offsets, the unpadded
    ones do not: hipFFT (iterated)."""
    tdt = _tdt()
    nx, ny, nz = dims
    rng = np.random.default_rng(nx)
    F = rng.standard_normal((nz, ny, nx))
    print(f"[case] padded rows {dims}", flush=True)
    s = tdt.Poisson3D(nx, ny, nz, 0.05, 0.06, 0.07, 0.3)
    U = to_host(s.solve(to_dev(F)))
    counts, _ = s.schedule()
    ref = P3.solve(F, 0.05, 0.06, 0.07, eps=0.3)
    _check_elementwise(U, ref, _tol(max(counts), _kappa(nx, ny, nz, 0.05, 0.06, 0.07)), f"{dims}")


def test_closed_form_has_no_line_bound():
    """The same bound does not refuse a grid in closed form (no line solves)."""
    print("[case] closed 3275 x 1023 x 1", flush=True)
    _tdt().Poisson3D(3275, 1023, 1, 0.05, 0.06, 0.07, 0.3)
