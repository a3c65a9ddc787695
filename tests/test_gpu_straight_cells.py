"""The default per-line kernel runs each cell as one straight stretch of
arithmetic and goes through it a second time, test by test, for the lanes
that failed some test in it; sets of more than 65,536 alive particles read the
parameters through scalar registers instead of LDS.  Both against the CPU
oracle, bit for bit, on operands that leave the drift's short sequences, on
losses in the first and last element of a cell, and on set sizes at the
edge between the two forms."""
import math

import numpy as np
import pytest

from paper_2310_00317_amd import inputs as I
from parity_util import assert_bitwise

pytestmark = pytest.mark.gpu
REF = I.PROTON_450GEV


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2310_00317_amd as P
    P.lib()
    return P


def _errored(order, seed):
    rng = np.random.default_rng(seed)
    scale = np.array([1e-7 * math.factorial(n) / 1e-2 ** n for n in range(order + 1)])
    return I.multipole(knl=rng.normal(0, 1, order + 1) * scale,
                       ksl=rng.normal(0, 1, order + 1) * scale)


def _line(kind):
    """Repeated cells of every element type; an odd piece at the end."""
    if kind == "apertures":    # a cell that starts and ends with a loss test
        cell = [I.ap_circle(0.02), I.multipole(knl=[0.0, 0.02]), I.drift(7.3),
                I.multipole(knl=[0.0, -0.02]), I.drift(7.3), I.ap_rect(-0.02, 0.021, -0.018, 0.02)]
    elif kind == "drifts":     # each class of drift length, tests in between
        cell = [I.drift(0.5), _errored(2, 1), I.drift(0.0), I.ap_ellipse(0.015, 0.012),
                I.drift(1.7), I.multipole(knl=[0.0, 5e-4]), I.drift(0.3, expanded=True),
                I.drift(-1.7), I.drift(2.0 ** -700), I.drift(0.7)]
    elif kind == "bends":      # curvature with and without a radiation length
        cell = [I.multipole(knl=[1e-4], hxl=1e-4, length=1.5), I.drift(2.0), _errored(10, 3),
                I.multipole(knl=[2e-4], hxl=2e-4), I.ap_circle(0.03), I.drift(1.1),
                I.multipole(knl=[0.0, 1e-3], length=0.7)]
    else:                      # frames and cavities
        cell = [I.xyshift(1e-4, -2e-4), I.srotation(0.1), _errored(1, 5), I.srotation(-0.1),
                I.xyshift(-1e-4, 2e-4), I.drift(1.5), I.rf(3e5, 4e8, 30.0), I.marker(),
                I.ap_circle(0.025), _errored(0, 6), I.drift(1.5)]
    return I.line(cell * 23 + cell[:3])


def _coords(n, seed):
    """A beam with losses, the hard cases scattered through it."""
    rng = np.random.default_rng(seed)
    c = rng.normal(0, [4e-3, 1e-4, 4e-3, 1e-4, 0.05, 1e-3], (n, 6))
    hard = np.array([
        [0, 0, 0, 0, 0, 0], [-0.0, -0.0, -0.0, -0.0, -0.0, -0.0],     # a drift numerator of zero
        [1e-170, 1e-170, 0, 0, 0, 0], [1e-3, 1e-95, 0, 0, 0, 0],      # underflowing squares
        [0, 0, 0, 0, 0, 1.5], [0, 0, 0, 0, 0, -0.9999999],            # momentum out of range
        [0, 0, 0, 0, 0, -1 + 1e-16], [0, 0, 0, 0, 0, 1e200],
        [0, 0.999, 0, 0.05, 0, 0], [0, 1.0, 0, 0, 0, 0], [0, 2.0, 0, 0, 0, 0],  # imaginary pz
        [0, 0, 0, 0, 0, -2.0 ** -53], [0, 0, 0, 0, 0, -2.0 ** -52],   # 1 + pz next to two
        [0, 2.0 ** -26, 0, 0, 0, 0], [0, 2.0 ** -25.5, 0, 2.0 ** -26, 0, 0],
        [0.02, 0, 0, 0, 0, 0], [np.nextafter(0.02, 1), 0, 0, 0, 0, 0],  # on the aperture's edge
        [np.nan, 0, 0, 0, 0, 0], [0, np.nan, 0, 0, 0, 0], [0, 0, 0, 0, np.nan, 0],
        [0, 0, 0, 0, 0, np.nan], [np.inf, 0, 0, 0, 0, 0], [0, 0, -np.inf, 0, 0, 0],
        [0, np.inf, 0, 0, 0, 0], [1e300, 0, 1e300, 0, 0, 0]])
    m = min(n, len(hard))
    at = rng.permutation(n)[:m]
    c[at] = hard[:m]
    return c


@pytest.mark.parametrize("kind", ["apertures", "drifts", "bends", "frames"])
@pytest.mark.parametrize("n", [1, 65, 1000, 65536, 65537, 70001])
def test_straight_cells_equal_the_oracle(P, oracle_mod, kind, n):
    el = _line(kind)
    # every hard case in the sets that hold them all; one in the set of one
    c = _coords(n, 7 + n)
    lat = P.Lattice(el, REF)
    parts = P.Particles(n, REF).init(c)
    # 1 + 2 turns: two chunks, the losses of the first compacted away, which
    # takes the largest sets below the edge between the forms
    passes, alive = P.track(lat, parts, 3, variant=14)
    g = parts.to_numpy()
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF)
        opasses = oracle_mod.track(el, REF, o, 3)
    assert_bitwise(g, o)
    assert passes == opasses and alive == int((o.state == 1).sum())
    if n >= 1000:   # the inputs exercise both outcomes
        assert 0.05 < np.mean(o.state == 1) < 0.999


@pytest.mark.parametrize("n", [1000, 70001])
def test_straight_cells_backward_and_batched(P, oracle_mod, n):
    el, el2 = _line("apertures"), _line("apertures")
    el2["knl"][el2["type"] == I.MULTIPOLE, 1] *= 1.01
    c = _coords(n, 3)
    lats = [P.Lattice(el, REF), P.Lattice(el2, REF)]
    parts = P.Particles(n, REF).init(c)
    P.track(lats[0], parts, 2, variant=14)
    P.track_backward(lats[0], parts, 2)
    with np.errstate(all="ignore"):
        o = oracle_mod.init(c, REF)
        oracle_mod.track(el, REF, o, 2)
        oracle_mod.track_backward(el, REF, o, 2)
    # the inverse maps negate the parameters, so the sign of a zero is free there
    plus = lambda d: {k: d[k] + 0.0 for k in ("x", "px", "y", "py", "zeta", "delta", "ptau")}  # noqa: E731
    g = parts.to_numpy()
    assert_bitwise(plus(g), plus(vars(o)), fields=tuple(plus(g)))
    assert_bitwise(g, o, fields=("state", "at_turn", "at_element"))
    # two variants, the boundary inside a wave
    cut = n // 2 + 5
    both = P.Particles(n, REF).init(c)
    P.track_batched(P.Batch(lats), both, [0, cut, n], 3, variant=14)
    g = both.to_numpy()
    for e, sl in ((el, slice(0, cut)), (el2, slice(cut, n))):
        with np.errstate(all="ignore"):
            o = oracle_mod.init(c[sl], REF)
            oracle_mod.track(e, REF, o, 3)
        assert_bitwise({k: v[sl] for k, v in g.items()}, o)
