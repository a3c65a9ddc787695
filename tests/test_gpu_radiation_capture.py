"""A caller's own capture of a radiation mode that the lattice has not tracked
yet, after another mode: the capture stays whole, and its replays give the eager
results."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from test_gpu_straight_cells import P  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.ELECTRON_45GEV6


@pytest.mark.parametrize("variant", [0, 14])
@pytest.mark.parametrize("first,mode", [(1, 2), (2, 1), (0, 2)])
def test_callers_capture(P, variant, first, mode):  # noqa: F811
    import torch
    n = 1000
    el = I.cfg5_lattice(100)
    c = I.cfg5_particles(n, 3)
    lat, eager_lat = P.Lattice(el, REF), P.Lattice(el, REF)
    P.track(lat, P.Particles(n, REF).init(c), 1, radiation=first, seed=5, variant=variant)
    parts = P.Particles(n, REF).init(c)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.track(lat, parts, 2, radiation=mode, seed=5, variant=variant, stats=False)
    for turns in (2, 4, 6):
        graph.replay()
        torch.cuda.synchronize()
        want = P.Particles(n, REF).init(c)
        P.track(eager_lat, want, turns, radiation=mode, seed=5)
        g, w = parts.to_numpy(), want.to_numpy()
        for f in ("x", "px", "y", "py", "zeta", "delta", "ptau", "state", "at_turn", "at_element"):
            assert np.array_equal(g[f], w[f]), (turns, f)
