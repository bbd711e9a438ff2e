"""Captured graphs for the GPU tests: their nodes counted (each kernel launch
is one), and replayed between eager work."""
import ctypes

import torch


def captured(fn):
    """fn() captured once (its buffers allocated before)."""
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        fn()
    g.instantiate()
    torch.cuda.synchronize()
    return g


def nodes(g) -> int:
    """Nodes of a captured graph."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    n = ctypes.c_size_t(0)
    status = ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None,
                                                ctypes.byref(n))
    assert status == 0, status
    return n.value


def replays_agree(g, outs, refs):
    """Three replays, with eager work and a synchronisation between, each leave
    refs in outs bit for bit."""
    for _ in range(3):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        if not all(torch.equal(o, r) for o, r in zip(outs, refs)):
            return False
    return True
