"""A caller's own capture of a call on more than 65,536 particles, on a lattice
that has tracked smaller sets only: the capture stays whole, and its replays
give the eager results."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from test_gpu_straight_cells import P, _line  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV


@pytest.mark.parametrize("built", [False, True])
def test_callers_capture(P, built):  # noqa: F811
    import torch
    n = 66001
    rng = np.random.default_rng(4)
    c = rng.normal(0, [1e-3, 1e-5, 1e-3, 1e-5, 0.02, 1e-4], (n, 6))
    lat = P.Lattice(_line("apertures"), REF)
    P.track(lat, P.Particles(100, REF).init(c[:100]), 1)
    eager_lat = P.Lattice(_line("apertures"), REF)
    if built:
        P.track(lat, P.Particles(n, REF).init(c), 1)
    parts = P.Particles(n, REF).init(c)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.track(lat, parts, 2, stats=False)
    assert P.wide_form(lat)[0] == int(built)
    for turns in (2, 4, 6):
        graph.replay()
        torch.cuda.synchronize()
        want = P.Particles(n, REF).init(c)
        P.track(eager_lat, want, turns)
        g, w = parts.to_numpy(), want.to_numpy()
        for f in ("x", "px", "y", "py", "zeta", "delta", "state", "at_turn", "at_element"):
            assert np.array_equal(g[f], w[f]), (turns, f)
    P.track(lat, P.Particles(n, REF).init(c), 1)
    assert P.wide_form(lat)[0] == 1
