"""Points on the spherical surface to the last digit: which are outside."""
from fractions import Fraction

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def fused(x, y):
    """x * x + y with one rounding"""
    return float(Fraction(x) * Fraction(x) + Fraction(y))


def test_points_on_the_sphere_are_judged_in_double_precision():
    """sqrt(x x + y y + z z) > radius with each product and sum rounded, as numpy has
    it: points of that distance within two digits of the radius, among them ones that
    fused products put on the other side."""
    import paper_2403_04053_amd as P
    n = (48, 48, 64)
    prob, _ = synth.tiny(n=n, P=4, transition=3, steps=2, dft=(0, 2))
    radius = 0.95
    prob = prob.replace(ramp_periods=0.0, tfsf=((16, 19, 29, 32), (16, 19, 29, 32), (24, 27, 37, 40)), surface_kind=1,
                        surf_lo=(14, 14, 22), surf_hi=(34, 34, 42), sphere_radius=radius, sphere_nodes=(4, 8))
    rng = np.random.default_rng(0)
    d = rng.normal(size=(4000, 3))
    d *= radius / np.linalg.norm(d, axis=1, keepdims=True)
    r = np.sqrt(d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1] + d[:, 2] * d[:, 2])
    other = np.array([np.sqrt(fused(p[2], fused(p[1], p[0] * p[0]))) for p in d])
    pick = np.concatenate([np.flatnonzero((r > radius) != (other > radius))[:40], np.arange(40)])
    assert ((r > radius) != (other > radius)).sum() >= 20
    s = P.Solver(prob)
    s.set_state(synth.random_state(n, 1), synth.random_state(n, 2), 0)
    s.run(1)
    for i in pick:
        try:
            s.project(d[i:i + 1])
            outside = True
        except P.PstdError as e:
            assert e.name == "PSTD_EINVAL"
            outside = False
        assert outside == bool(r[i] > radius), (i, r[i])
    s.close()
