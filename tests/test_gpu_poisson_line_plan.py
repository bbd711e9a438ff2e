"""The line plan of a 2D Poisson handle whose modes are solved in place: asking
for it and reading its profile change neither the solves nor graphs captured
before; launch options move the solves to the plan that has them, and their
defaults move them back.

99 and 100: mixed-radix and matrix transforms (100 and 101 intervals); 2000
rows: tiled columns with a workspace of their own."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host
from oracle import poisson2d as P2
from test_gpu_poisson import tol as tol2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [300, 2000])
@pytest.mark.parametrize("nx", [99, 100])
def test_line_plan_leaves_the_solves_alone(nx, ny):
    import torch

    import paper_1002_2469_amd as tdt
    from gpu_graph import captured, nodes, replays_agree
    rng = np.random.default_rng(nx)
    hx, hy = 0.01, 0.004
    Fh = rng.standard_normal((ny, nx))
    F = to_dev(Fh)
    U = torch.empty_like(F)
    print(f"[case] line plan {nx} x {ny}", flush=True)
    s = tdt.Poisson2D(nx, ny, hx, hy)
    U0 = s.solve(F).clone()
    ref = P2.solve(Fh, hx, hy)
    assert oracle.rel_err(to_host(U0), ref) <= tol2(nx, ny, hx, hy)
    g = captured(lambda: s.solve(F, U))
    n0 = nodes(g)

    s.line_profile(True)
    assert torch.equal(s.solve(F), U0)
    read = s.line_profile_read()
    assert read["solves"] == 1 and read["final_ms"] > 0.0
    assert nodes(captured(lambda: s.solve(F, U))) == n0
    assert replays_agree(g, [U], [U0])
    s.line_profile(False)

    s.set_line_option("whole_max_tiles", 0)
    assert oracle.rel_err(to_host(s.solve(F)), ref) <= tol2(nx, ny, hx, hy)
    assert nodes(captured(lambda: s.solve(F, U))) > n0
    assert replays_agree(g, [U], [U0])   # (the graph of the in-place solve)
    s.line_profile(True)
    s.solve(F)
    assert s.line_profile_read()["solves"] == 1

    s.set_line_option("whole_max_tiles", 8)
    assert torch.equal(s.solve(F), U0)
    assert nodes(captured(lambda: s.solve(F, U))) == n0
    assert replays_agree(g, [U], [U0])


def test_line_plan_of_a_power_of_two():
    """The strided plan itself, which takes no options."""
    import paper_1002_2469_amd as tdt
    s = tdt.Poisson2D(127, 40, 0.01, 0.02)
    print("[case] line plan 127 x 40", flush=True)
    F = to_dev(np.random.default_rng(1).standard_normal((40, 127)))
    s.line_profile(True)
    s.solve(F)
    assert s.line_profile_read()["solves"] == 1
    with pytest.raises(Exception):
        s.set_line_option("whole_max_tiles", 0)
