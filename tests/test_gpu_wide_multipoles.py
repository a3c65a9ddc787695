"""Several high-order multipoles in a row, more parameter words than there are
scalar registers, in the form for more than 65,536 alive particles: spilled
words come back just before the multiply-adds that read them.  Bit for bit
against the CPU oracle."""
import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from parity_util import assert_bitwise
from test_gpu_straight_cells import P, _coords, _errored  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV
DRIFT, APERTURE = I.drift(1.3), I.ap_circle(0.03)
CELLS = {
    "7-7-7": [_errored(7, 1), _errored(7, 2), _errored(7, 3), DRIFT, APERTURE],
    "10-10-10": [_errored(10, 1), _errored(10, 2), _errored(10, 3), DRIFT],
    "10-bend-10": [_errored(10, 1), I.multipole(knl=[1e-4, 1e-3], hxl=1e-4, length=1.5),
                   _errored(10, 2), DRIFT, APERTURE],
    "10-cavity-10-9": [_errored(10, 1), I.rf(3e5, 4e8, 30.0), _errored(10, 2), _errored(9, 3),
                       DRIFT, APERTURE],
    "5-10-5": [_errored(5, 1), _errored(10, 2), _errored(5, 3), DRIFT],
}


@pytest.mark.parametrize("cell", list(CELLS))
@pytest.mark.parametrize("n", [65, 66001])
def test_multipoles_in_a_row(P, oracle_mod, cell, n):  # noqa: F811
    el = I.line(CELLS[cell] * 20)
    c = _coords(n, 5)
    parts = P.Particles(n, REF).init(c)
    passes, alive = P.track(P.Lattice(el, REF), parts, 2, variant=14)
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF)
        opasses = oracle_mod.track(el, REF, o, 2)
    assert_bitwise(parts.to_numpy(), o)
    assert passes == opasses and alive == int((o.state == 1).sum())
    if n > 65536:
        assert alive > 0


def test_batch_of_multipoles_in_a_row(P, oracle_mod):  # noqa: F811
    n, cut = 66001, 33005
    els = [I.line([_errored(10, s), _errored(10, s + 1), APERTURE, DRIFT] * 20) for s in (1, 7)]
    c = _coords(n, 6)
    parts = P.Particles(n, REF).init(c)
    batch = P.Batch([P.Lattice(e, REF) for e in els])
    P.track_batched(batch, parts, np.array([0, cut, n], dtype=np.int64), 2, variant=14)
    g = parts.to_numpy()
    for e, sl in ((els[0], slice(0, cut)), (els[1], slice(cut, n))):
        with np.errstate(all="ignore"):
            o = oracle_mod.init(c[sl], REF)
            oracle_mod.track(e, REF, o, 2)
        assert_bitwise({k: v[sl] for k, v in g.items()}, o)
