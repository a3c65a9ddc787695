"""Radiating multipoles inside the default kernel's straight cells: the short
sequences of the radiation step and of the bend's curvature term, and the
second pass through a cell for operands that they do not serve, bit for bit
against the CPU oracle; the lines and states that the kernel leaves to the
general operations give the same values as the branching form."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from parity_util import assert_bitwise
from test_gpu_straight_cells import P, _coords  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.ELECTRON_45GEV6


def _line(kind):
    bend = I.multipole(knl=[2e-3, 1e-3], hxl=2e-3, length=9.3)
    if kind == "bends":
        cell = [I.multipole(knl=[0.0, 0.02]), I.drift(3.1), I.multipole(knl=[1e-3], hxl=1e-3, length=8.0),
                I.ap_circle(0.3), I.drift(3.1), bend, I.multipole(knl=[0.0, -0.02]), I.drift(1.7)]
    elif kind == "lengths":   # radiation without curvature, no kick at all, all-ones lengths
        ones = float(np.nextafter(8.0, 0))
        cell = [I.multipole(knl=[0.0, 0.02], length=0.7), I.drift(2.5),
                I.multipole(knl=[0.0], length=1.0), I.multipole(knl=[1e-3], hxl=1e-3, length=ones),
                I.drift(2.5), I.multipole(knl=[0.0, -0.02], length=ones), I.rf(5e6, 4e8, 30.0),
                I.ap_rect(-0.3, 0.3, -0.3, 0.3), I.drift(0.7)]
    else:                     # a length and a curvature that the short sequences do not serve
        cell = [bend, I.drift(2.5), I.multipole(knl=[1e-4], hxl=1e-4), I.drift(1.5),
                I.multipole(knl=[1e-4], hxl=2.0 ** -120, length=2.0), I.ap_circle(0.3)]
    return I.line(cell * 17 + cell[:3])


@pytest.mark.parametrize("kind", ["bends", "lengths", "unserved"])
@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("n", [1, 65, 1000, 66001])
def test_radiation_in_straight_cells(P, oracle_mod, kind, mode, n):  # noqa: F811
    el = _line(kind)
    c = _coords(n, 11 + n)
    lat = P.Lattice(el, REF)
    parts = P.Particles(n, REF).init(c, first_id=(1 << 32) - 3)
    passes, alive = P.track(lat, parts, 3, radiation=mode, seed=77, variant=14)
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF, first_id=(1 << 32) - 3)
        opasses = oracle_mod.track(el, REF, o, 3, radiation=mode, seed=77)
    assert_bitwise(parts.to_numpy(), o)
    assert passes == opasses and alive == int((o.state == 1).sum())
    if n >= 1000:
        assert 0.05 < np.mean(o.state == 1) < 0.999


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_state_not_from_init(P, oracle_mod, mode):  # noqa: F811
    """A caller's own rpp (not the rounded 1/(1+delta)) and positions beyond
    the curvature term's short division: as the branching form."""
    import torch
    c = _coords(500, 5)
    out = []
    for variant in (10, 14):
        lat = P.Lattice(_line("bends"), REF)
        parts = P.Particles(500, REF).init(c)
        parts.rpp[::3] *= 1.0 + 1e-12
        parts.x[7], parts.x[8], parts.x[9] = 1e200, -0.0, 1e-250
        P.track(lat, parts, 2, radiation=mode, seed=5, variant=variant)
        out.append(parts.to_numpy())
    assert_bitwise(out[1], out[0])
    torch.cuda.synchronize()


@pytest.mark.parametrize("mode", [1, 2])
def test_radiating_batch(P, oracle_mod, mode):  # noqa: F811
    """Two variants as one batch, above and below the form for large sets."""
    el, el2 = _line("bends"), _line("bends")
    el2["knl"][el2["hxl"] != 0, 0] *= 1.01
    lats = [P.Lattice(el, REF), P.Lattice(el2, REF)]
    for n in (700, 66001):
        c, cut = _coords(n, 3), n // 2 + 5
        both = P.Particles(n, REF).init(c)
        P.track_batched(P.Batch(lats), both, np.array([0, cut, n], dtype=np.int64), 2,
                        radiation=mode, seed=4, variant=14)
        g = both.to_numpy()
        for e, a, b in ((el, 0, cut), (el2, cut, n)):
            with np.errstate(all="ignore"):
                o = oracle_mod.init(c[a:b], REF, first_id=a)
                oracle_mod.track(e, REF, o, 2, radiation=mode, seed=4)
            assert_bitwise({k: v[a:b] for k, v in g.items()}, o)
