"""Rounding of the box far field against 80-bit sums of the cell formula's factors."""
import math

import numpy as np
import pytest

import synth
from oracle import pstd as opstd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LD, CLD = np.longdouble, np.clongdouble
PI = 4 * np.arctan(LD(1))


def expi(x):
    return np.cos(x) + 1j * np.sin(x).astype(CLD)


def factor(N, lo, hi, d, r):
    """h[i]: what the plane value at grid index i contributes along one axis, the
    trigonometric interpolant of the cells [lo, hi) times exp(-i r x), integrated."""
    m = np.arange(N)
    b = np.where(m < N // 2, m, m - N)
    theta = PI * b / LD(N) - d * r / 2
    n = hi - lo
    small = np.abs(theta) < LD(1e-30)
    t = np.where(small, 1, theta)
    mag = np.where(small, LD(n), np.sin(n * theta) / t) * np.where(b & 1, -1, 1)
    # sum of exp(2 i theta (l - N/2 + 1/2)) about its middle
    g = mag * expi(theta * LD(lo + hi - N))
    w = expi(-2 * PI * ((m[:, None] * m[None, :]) % N) / LD(N))
    return (g[:, None] * w).sum(0)


def far_field(prob, dxb, phi, dphi, dirs):
    out = []
    dxb = [LD(x) for x in dxb]
    for v in dirs:
        r = [LD(x) for x in v]
        h = [factor(prob.n[a], prob.surf_lo[a], prob.surf_hi[a], dxb[a], r[a]) for a in range(3)]
        f = CLD(0)
        for face in range(6):
            a, side = divmod(face, 2)
            b, c = (1, 2) if a == 0 else (0, 2) if a == 1 else (0, 1)
            xa = ((prob.surf_hi if side else prob.surf_lo)[a] - prob.n[a] // 2) * dxb[a]
            plane = dphi[face].astype(CLD) + 1j * r[a] * phi[face].astype(CLD)
            s = ((plane * h[b][None, :]).sum(1) * h[c]).sum()
            f += (-1 if side else 1) * dxb[b] * dxb[c] / (prob.n[b] * prob.n[c]) * s * expi(-r[a] * xa)
        out.append(f / (4 * PI * LD(prob.k0)))
    return np.array(out)


@pytest.mark.parametrize("n,ppw", [((160, 160, 160), 8), ((64, 96, 108), 8), ((288, 48, 64), 3)])
def test_far_field_rounding(n, ppw):
    """RMS error over 64 directions of a field of random planes, u = 2^-53, X the
    largest reduced half width of the box.  A direction's angle is rounded once, by
    at most u |a|, uniformly: u |a| / sqrt(3) RMS, and moves the phases of cells whose
    positions have the RMS X / sqrt(3), by cos a: under u X / 4.  The transforms and the
    two sums of some hundred products each, errors adding like a random walk: 16 u.
    (Chebyshev nodes taken as their rounded values add u X / 3 at least.)"""
    import paper_2403_04053_amd as P
    prob, _ = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=1, dft=(0, 1))
    h = 2 * math.pi / (ppw * prob.k0)
    prob = prob.replace(h=(h, h, h), ramp_periods=0.0, theta=0.6, phi=0.9)
    s = P.Solver(prob)
    s.set_state(synth.random_state(n, 1), synth.random_state(n, 2), 0)
    s.run(1)
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    g = np.random.default_rng(11).normal(size=(64, 3))
    dirs = g / np.linalg.norm(g, axis=1, keepdims=True)
    got = s.far_field(dirs).cpu().numpy()
    want = far_field(prob, opstd.dxbar(prob), phi, dphi, dirs)
    rms = lambda x: math.sqrt(float((np.abs(x) ** 2).mean()))
    err = rms(got.astype(CLD) - want) / rms(want)
    X = max((prob.surf_hi[a] - prob.surf_lo[a]) * opstd.dxbar(prob)[a] / 2 for a in range(3))
    bound = 2.0 ** -53 * (X / 4 + 16)
    print(f"far field {n}, {ppw} points per wavelength: RMS error {err:.2e}, bound {bound:.2e}", flush=True)
    s.close()
    assert err <= bound
