"""The end of a chunk in one launch for sets of at most 1,024 particles and in
two above: alive list, pass count and turn, with and without compaction, for
the interpreter (which replays the chunk's losses from the turn the chunk
started at) and the default kernel, forward, backward and from a graph."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from parity_util import assert_bitwise
from test_gpu_straight_cells import P, _coords, _line  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 3000])
@pytest.mark.parametrize("variant", [4, 14])
@pytest.mark.parametrize("compact", [True, False])
def test_chunks(P, oracle_mod, n, variant, compact):  # noqa: F811
    el = _line("apertures")
    c = _coords(n, 2)
    lat = P.Lattice(el, REF)
    parts = P.Particles(n, REF).init(c)
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF)
        for turns, kw in ((5, dict(turns_per_chunk=2)), (3, {}), (4, dict(graph=True))):
            got = P.track(lat, parts, turns, variant=variant, compact=compact, **kw)
            want = oracle_mod.track(el, REF, o, turns)
            assert got[0] == want, (turns, kw)
            if compact:   # (without, the list keeps its length)
                assert got[1] == int((o.state == 1).sum()), (turns, kw)
            assert_bitwise(parts.to_numpy(), o)
        P.track(lat, parts, 2, variant=variant, compact=compact, stats=False)
        oracle_mod.track(el, REF, o, 2)
        got = P.track_backward(lat, parts, 3)
        want = oracle_mod.track_backward(el, REF, o, 3)
    if compact:   # (an uncompacted list counts the turns of its earlier losses again)
        assert got == (want, int((o.state == 1).sum()))
    assert_bitwise(parts.to_numpy(), o, fields=("state", "at_turn", "at_element"))
    assert parts.turn == 5 + 3 + 4 + 2 - 3


def test_empty_set(P, oracle_mod):  # noqa: F811
    lat = P.Lattice(_line("drifts"), REF)
    parts = P.Particles(0, REF).init(np.zeros((0, 6)))
    assert P.track(lat, parts, 3) == (0, 0) and parts.turn == 3
