"""Kernels per call, counted as the nodes of a captured graph."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1406_4350_amd import chebfd as cf  # noqa: E402
from paper_1406_4350_amd import workload as wl  # noqa: E402


def _nodes(fn):
    """Nodes of the graph that fn's launches on a stream of its own make (fn has run once before)."""
    hip = ctypes.CDLL("libamdhip64.so")
    fn()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(s):
        st = ctypes.c_void_p(s.cuda_stream)
        assert hip.hipStreamBeginCapture(st, 2) == 0
        fn()
        assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("nb", [1, 41, 64])
def test_single_operators_take_no_reduction_launch(nb):
    """24^3, 925 plane waves, 65 projectors: projection, projector space, back-projection (and three transforms for H)."""
    pb = wl.make_problem(wl.Config("launches24", 24, 6, 6.0, "random", 1, 5, "2s2p1d", True, nb, 4, 1, 1, 171))
    plan = cf.plan_from_problem(pb, cf.CHEB_FP64)
    X = torch.randn((nb, pb.npw), dtype=torch.complex128, device="cuda")
    Y = torch.empty_like(X)
    assert _nodes(lambda: plan.apply_S(X, Y)) == 3
    assert _nodes(lambda: plan.apply_Sinv(X, Y)) == 3
    assert _nodes(lambda: plan.apply_H(X, Y)) == 6
    plan.close()
