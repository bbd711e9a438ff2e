"""An iterated 3D solve whose padded rows do not fit the device any more takes
the unpadded ones (Nx = 1: 64 doubles of workspace per row padded, 6 not), as
it did before rows were padded there."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from oracle import poisson3d as P3
from test_gpu_poisson3d import _check_elementwise, _kappa, _tol

pytestmark = pytest.mark.gpu


def test_unpadded_rows_when_memory_is_short():
    import torch

    import paper_1002_2469_amd as tdt
    nx, ny, nz, h = 1, 1500, 1500, (0.05, 0.06, 0.07)
    F = np.random.default_rng(2).standard_normal((nz, ny, nx))
    Fd = to_dev(F)
    tdt.Poisson3D(3, 20, 1100, *h, 0.3).solve(torch.zeros(1100, 20, 3, dtype=torch.float64,
                                                          device=Fd.device))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    print("[case] 3D unpadded rows, little memory", flush=True)
    # all but a little: one large block, 400 MiB ones until none is left, less one
    free, _ = torch.cuda.mem_get_info()
    held = [torch.empty(max(1, free - (8 << 30)), dtype=torch.uint8, device=Fd.device)]
    try:
        for _ in range(100):
            held.append(torch.empty(400 << 20, dtype=torch.uint8, device=Fd.device))
    except torch.OutOfMemoryError:
        pass
    held.pop()
    torch.cuda.empty_cache()
    try:
        s = tdt.Poisson3D(nx, ny, nz, *h, 0.3)   # (padded: 2 x 549 MiB)
        U = to_host(s.solve(Fd))
        counts, _ = s.schedule()
        s.close()
    finally:
        held.clear()
        torch.cuda.empty_cache()
    ref = P3.solve(F, *h, eps=0.3)
    _check_elementwise(U, ref, _tol(max(counts), _kappa(nx, ny, nz, *h)), "short memory")
