"""The Fresnel projection's series on grids of unequal and coarse spacings, against
series of an order at which they are exact to rounding."""
import math

import numpy as np
import pytest

import synth
from oracle import adjoint as oadj
from oracle import ntdf as ontdf
from oracle import pstd as opstd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ORDER = 20  # of the reference: a^21 / 22! is 1e-20 at 3 points per wavelength


def spaced(n, ppw, **kw):
    """The small geometry with its own number of points per wavelength on each axis."""
    kw = dict(dict(transition=2, v0=0.5, theta=0.6, phi=0.9), **kw)
    prob, V = synth.tiny(n=n, P=3, radius_cells=2, **kw)
    return prob.replace(h=tuple(2 * math.pi / (p * prob.k0) for p in ppw)), V


def series_bound(prob):
    """The 9th-order terms of the two largest spacings, each at most a^9 / 10!, twice:
    what the 8th-order series drop and what the economised terms leave."""
    a = np.sort(np.asarray(opstd.dxbar(prob)) / 2)[1:]
    return 2 * float((a ** 9).sum()) / math.factorial(10)


def economised_bound(prob):
    """What the economised terms may leave of the 81 products of a face's two series,
    the largest over the faces: of the largest value of each monomial of degree 9 and 10
    on the disk a tenth, of degree 11 to 16 a fifth (1/11 and 1/5.4 measured), times the
    series' coefficients, at most 1 / ((p + 1)! (q + 1)!)."""
    a = np.asarray(opstd.dxbar(prob)) / 2
    worst = 0.0
    for b, c in ((0, 1), (0, 2), (1, 2)):
        s = 0.0
        for p in range(1, 9):
            for q in range(9 - p, 9):
                top = math.sqrt(p ** p * q ** q / (p + q) ** (p + q))
                s += (0.1 if p + q < 11 else 0.2) * top * a[b] ** p * a[c] ** q / (math.factorial(p + 1) *
                                                                                   math.factorial(q + 1))
        worst = max(worst, s)
    return worst


@pytest.mark.parametrize("n,ppw", [((24, 20, 32), (8, 8, 8)), ((24, 20, 32), (8, 5, 12)), ((24, 20, 32), (3, 4, 6)),
                                   ((20, 32, 24), (6, 3, 3.5)), ((32, 24, 20), (12, 4, 3)), ((24, 20, 32), (3, 12, 4)),
                                   ((20, 24, 32), (4, 3, 12))])
def test_points_with_three_spacings(n, ppw):
    """Random planes: the sincs of a cell's modes are 0.4 (edge of the spectrum on both
    axes) to 1, and their errors add up as the modes do, so the relative error of the sum
    is at most 2.5 times that of the series, 4 at the largest of a few points; rounding
    1e-13.  Against exact series, and against the 8th-order ones, which the economised
    terms stand for.  (With the two half widths exchanged the last three are off by 9
    times the second bound.)"""
    import paper_2403_04053_amd as P
    prob, _ = spaced(n, ppw, steps=1, dft=(0, 1))
    prob = prob.replace(ramp_periods=0.0)
    s = P.Solver(prob)
    s.set_state(synth.random_state(n, 1), synth.random_state(n, 2), 0)
    s.run(1)
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    box = ontdf.Box(prob.n, opstd.dxbar(prob), prob.surf_lo, prob.surf_hi)
    half = np.array([(prob.surf_hi[a] - prob.surf_lo[a]) * prob.h[a] / 2 for a in range(3)])
    rng = np.random.default_rng(7)
    pts = rng.uniform(-1, 1, size=(24, 3))
    pts /= np.abs(pts).max(1, keepdims=True)
    pts *= half * rng.uniform(1.15, 3.0, size=(24, 1))
    got = s.project(pts).cpu().numpy()
    s.close()
    for order, bound in ((ORDER, series_bound(prob)), (8, economised_bound(prob))):
        want = ontdf.TaylorTables(box, phi, dphi, order=order).project(pts * prob.k0)
        err = np.abs(got - want).max() / np.abs(want).max()
        print(f"points, {ppw} points per wavelength, order {order}: {err:.2e}, bound {4 * bound + 1e-13:.2e}", flush=True)
        assert err <= 4 * bound + 1e-13


def test_gradient_with_three_spacings():
    """The misfit and its gradient, whose projection and adjoint take the same series,
    next to whose errors (4e-8) those of the FP32 steps stand: phasors to about 2e-5,
    twice that in an intensity, twice again in the square of its difference from the
    target, half as large: 5e-4 with a few points; the gradient as on equal spacings,
    1e-3."""
    import paper_2403_04053_amd as P
    steps = 60
    prob, V = spaced((20, 24, 32), (6, 4, 9), steps=steps, dft=(20, steps), transition=3, v0=1.5, theta=0.0, phi=0.0)
    prob = prob.replace(ramp_periods=0.5)
    V = V.astype(np.float32).astype(np.float64)
    half = np.array([(prob.surf_hi[a] - prob.surf_lo[a]) * prob.h[a] / 2 for a in range(3)])
    pts = np.vstack([np.eye(3), -np.eye(3), [[1, 1, 1]], [[-1, 0.5, 1]]]) * half * 1.4
    target = oadj.intensity(prob, 0.5 * V, pts, order=14)
    J_ref, g_ref = oadj.gradient(prob, V, pts, target, order=14)
    s = P.Solver(prob)
    s.set_potential(V)
    J = s.misfit(steps, pts, target)
    g = s.misfit_gradient().cpu().numpy().astype(np.float64)
    err = np.linalg.norm(g - g_ref) / np.linalg.norm(g_ref)
    print(f"misfit {J_ref:.3e} {abs(J - J_ref) / J_ref:.2e}, gradient {err:.2e}", flush=True)
    s.close()
    assert abs(J - J_ref) <= 5e-4 * J_ref
    assert err <= 1e-3
