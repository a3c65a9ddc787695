"""The second form of the default kernel, for more than 65,536 alive particles,
is there and is launched: the tests of those sizes compare results, which the
other form gives as well."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from test_gpu_straight_cells import P, _line  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV


def _set(P, n):  # noqa: F811
    c = np.zeros((n, 6))
    c[:, 0] = np.linspace(-1e-3, 1e-3, n)
    return P.Particles(n, REF).init(c)


@pytest.mark.parametrize("kind", ["apertures", "drifts", "bends", "frames"])
def test_lattice(P, kind):  # noqa: F811
    lat = P.Lattice(_line(kind), REF)
    assert P.wide_form(lat) == (0, 0, "")
    P.track(lat, _set(P, 65536), 3)
    assert P.wide_form(lat) == (0, 0, "")
    P.track(lat, _set(P, 65537), 6, turns_per_chunk=2)
    assert P.wide_form(lat) == (1, 3, "")
    P.track(lat, _set(P, 65537), 2, turns_per_chunk=1, graph=True)
    P.track_backward(lat, _set(P, 65537), 1)
    state, launches, _ = P.wide_form(lat)
    assert state == 1 and launches == 5
    assert P.wide_form(lat, backward=True)[:2] == (1, 1)


def test_radiation_has_none(P):  # noqa: F811
    lat = P.Lattice(_line("bends"), REF)
    P.track(lat, _set(P, 65537), 1, radiation=1)
    assert P.wide_form(lat) == (0, 0, "")


def test_batch(P):  # noqa: F811
    batch = P.Batch([P.Lattice(_line("apertures"), REF) for _ in range(2)])
    P.track_batched(batch, _set(P, 65537), np.array([0, 9, 65537], dtype=np.int64), 2,
                    turns_per_chunk=1)
    assert P.wide_form(batch) == (1, 2, "")
