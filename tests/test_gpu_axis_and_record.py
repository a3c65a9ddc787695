"""The recording kernel of optics by tracking, whose cells are straight and
whose parameters a second wave brings ahead, on lines of fewer cells than that
wave's lead, on operands that leave the short sequences and on particle counts
around a workgroup; and the reference particle on the axis, which the straight
cells serve where the line keeps it there.  Bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from parity_util import assert_bitwise
from test_gpu_straight_cells import P, _coords, _line  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV


@pytest.mark.parametrize("kind", ["apertures", "drifts", "bends", "frames"])
@pytest.mark.parametrize("n,elements", [(1, 1), (1, 7), (63, 12), (64, 60), (65, 130), (130, 231)])
def test_record(P, oracle_mod, kind, n, elements):  # noqa: F811
    el = _line(kind)[:elements].copy()
    c = _coords(n, 21 + n)
    g = P.track_record(P.Lattice(el, REF), c).cpu().numpy()
    with np.errstate(all="ignore"):
        o = oracle_mod.track_record(el, REF, c)
    same = (g.view(np.int64) == o.view(np.int64)) | (np.isnan(g) & np.isnan(o))
    assert same.all(), f"{(~same).sum()} values differ"


def _axis_line(kind):
    if kind == "kept":       # no kick on the axis, a bend whose curvature takes its kick back
        cell = [I.multipole(knl=[0.0, 0.02]), I.drift(2.3), I.multipole(knl=[1e-3, 2e-4], hxl=1e-3,
                length=4.7), I.drift(2.3), I.multipole(knl=[0.0, -0.02, 0.3]), I.drift(1.7),
                I.multipole(knl=[2e-3], hxl=2e-3)]
    elif kind == "cavity":   # the momentum changes at every turn
        cell = [I.multipole(knl=[0.0, 0.02]), I.drift(2.3), I.rf(3e5, 4e8, 30.0), I.drift(1.7)]
    elif kind == "still":    # a cavity that leaves the momentum of zeta = 0 alone
        cell = [I.multipole(knl=[0.0, 0.02]), I.drift(2.3), I.rf(3e5, 4e8, 0.0), I.drift(1.7)]
    else:                    # kicks and shifts so small that the drifts' numerators underflow
        k = 2.0 ** {"kicks": -310, "shifts": -20}[kind]
        cell = ([I.multipole(knl=[k]), I.drift(2.3), I.multipole(knl=[-2 * k, 0.01]), I.drift(2.3),
                 I.multipole(knl=[k])] if kind == "kicks" else
                [I.xyshift(k, 0.0), I.multipole(knl=[0.0, 0.02]), I.drift(2.3),
                 I.xyshift(-k, 0.0), I.drift(2.3)])
    return I.line(cell * 19 + cell[:2])


@pytest.mark.parametrize("kind", ["kept", "cavity", "still", "kicks", "shifts"])
@pytest.mark.parametrize("n", [70, 66001])
def test_reference_particle(P, oracle_mod, kind, n):  # noqa: F811
    el = _axis_line(kind)
    c = np.random.default_rng(3).normal(0, [1e-4, 1e-6, 1e-4, 1e-6, 0.02, 1e-4], (n, 6))
    c[:16] = 0.0
    c[1] = -0.0
    c[2, 5], c[3, 5], c[4, 4] = -0.0, 1e-200, 0.01
    c[5, 1], c[6, 1], c[7, 0], c[8, 5] = 1e-170, 1e-150, 1e-160, 1e-3
    lat = P.Lattice(el, REF)
    parts = P.Particles(n, REF).init(c)
    P.track(lat, parts, 3, variant=14)
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF)
        oracle_mod.track(el, REF, o, 3)
    assert_bitwise(parts.to_numpy(), o)
    g = P.track_record(lat, c[:64]).cpu().numpy()
    r = oracle_mod.track_record(el, REF, c[:64])
    same = (g.view(np.int64) == r.view(np.int64)) | (np.isnan(g) & np.isnan(r))
    assert same.all(), f"{(~same).sum()} values differ"
