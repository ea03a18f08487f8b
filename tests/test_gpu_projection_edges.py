"""GPU parity of the projection kernels at the edges of their launch shapes
(counts that leave part of a workgroup, wave or split idle), against the FP64
oracle on the same phasors."""
import math

import numpy as np
import pytest

import synth
from oracle import ntdf as ontdf
from oracle import pstd as opstd
from oracle import sphere as osph

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available()
    import paper_2403_04053_amd as mod
    return mod


def sphere_case(P, nodes, seed=0):
    """A 48 x 48 x 64 solver whose shell sums are a given field (one window
    step from a seeded state, no switch-on), and the oracle's node phasors."""
    h = 0.1
    k0 = 2 * math.pi / (8 * h)
    xy, z = (16, 19, 29, 32), (24, 27, 37, 40)
    prob = synth.Problem(n=(48, 48, 64), h=(h,) * 3, k0=k0, theta=0.5, phi=0.8, abc_cells=(4,) * 3, abc_alpha=1.0,
                         abc_U0=5.0, tfsf=(xy, xy, z), v_max=0.5 * k0 * k0 / 2, ramp_periods=0.0, n_steps=1,
                         dft_begin=0, dft_end=1, surf_lo=(14, 14, 22), surf_hi=(34, 34, 42), surface_kind=1,
                         sphere_radius=0.95, sphere_nodes=nodes)
    field = synth.random_state(prob.n, seed).astype(np.complex64)
    s = P.Solver(prob)
    s.set_state(np.zeros_like(field), field, 0)
    s.run(1)
    sph = osph.Sphere(prob, prob.sphere_radius, n_theta=nodes[0], n_phi=nodes[1])
    m = opstd.build(prob, np.zeros((prob.n[2], prob.n[1], prob.n[0])))
    ref = sph.node_values(field.astype(np.complex128) - m.zeta * m.phase)
    return s, sph, ref


@pytest.mark.parametrize("nodes", [(2, 3), (3, 7), (16, 32)])
def test_node_phasors_of_a_given_field(P, nodes):
    """Node counts that leave waves of the last workgroup idle.  Sums of 512
    FP64 terms against the oracle's: 512 roundings of 2^-53 each, so 1e-12 of
    the largest phasor."""
    s, _, (rv, rd) = sphere_case(P, nodes)
    v, d = (x.cpu().numpy() for x in s.sphere_phasors())
    assert np.abs(v - rv).max() <= 1e-12 * np.abs(rv).max()
    assert np.abs(d - rd).max() <= 1e-12 * np.abs(rd).max()


def box_case(P, n, steps=200):
    prob, V = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=steps, theta=0.4, phi=1.0)
    prob = prob.replace(ramp_periods=0.5, dft_begin=steps // 2, dft_end=steps)
    s = P.Solver(prob)
    s.set_potential(V)
    s.run(steps)
    return prob, s, ontdf.Box(prob.n, opstd.dxbar(prob), prob.surf_lo, prob.surf_hi)


def directions(count, seed=0):
    d = np.random.default_rng(seed).normal(size=(count, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True)


@pytest.mark.parametrize("n", [(24, 20, 32), (40, 24, 20), (64, 48, 24)])
@pytest.mark.parametrize("count", [1, 15, 17, 64, 65, 300])
def test_box_far_field_counts(P, n, count):
    """Direction counts that leave waves and their lanes idle, the poles and
    the axes among them, on boxes with odd and even numbers of Chebyshev terms.
    Series cut at 2^-57 and a few hundred FP64 additions: 1e-12 of the largest."""
    prob, s, box = box_case(P, n)
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    d = directions(count)
    special = np.array([[0, 0, 1.0], [0, 0, -1.0], [1.0, 0, 0], [0, -1.0, 0]])
    d[:min(4, count)] = special[:count]
    got = s.far_field(d).cpu().numpy()
    ref = ontdf.far_field(box, phi, dphi, d) / prob.k0
    big = ontdf.far_field(box, phi, dphi, directions(20, 1)) / prob.k0
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(big).max()


def test_box_far_field_of_vectors_beyond_unit_length(P):
    """The formula holds for any vector; components beyond 1 lie outside the
    series' interval and take the direct sums (one among many unit vectors, in
    a second group of 256)."""
    prob, s, box = box_case(P, (24, 20, 32))
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    d = directions(600)
    d[3] *= 2.5
    d[400] = (0.0, 1.5, -0.3)
    d[599] = (0.2, -0.3, 1.0000001)
    got = s.far_field(d).cpu().numpy()
    ref = ontdf.far_field(box, phi, dphi, d) / prob.k0
    assert np.all(np.abs(got - ref) <= 1e-11 * np.maximum(np.abs(ref), np.abs(ref).max() * 1e-3))
    assert torch.isnan(torch.view_as_real(s.far_field(np.array([[np.nan, 0.0, 0.0]])))).all()


@pytest.mark.parametrize("n", [(24, 20, 32), (40, 24, 20)])
@pytest.mark.parametrize("count", [1, 255, 257, 513])
def test_box_points_counts(P, n, count):
    """Point counts around the workgroup's 2 x 256, close points (the largest
    cell angles) among them, against the 8th-order series of the oracle; the economised terms differ from it by
    under 1/50 of the degree-9 terms, a^9 / 10! with a <= pi/8: 1e-11 of the largest."""
    prob, s, box = box_case(P, n)
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    h = prob.h[0]
    half = [(prob.surf_hi[a] - prob.surf_lo[a]) * h / 2 for a in range(3)]
    pts = directions(count, 2) * np.random.default_rng(3).uniform(1.8, 6.0, size=(count, 1)) * max(half)
    if count > 2:
        pts[0] = (half[0] + 0.05, 0.02, -0.03)
        pts[1] = (0.1, -(half[1] + 0.3), 0.0)
    tab = ontdf.TaylorTables(box, phi, dphi)
    ref = tab.project(pts * prob.k0)
    got = s.project(pts).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
    # a point beyond the short sincos's range sends all through the general one
    far = np.vstack([pts[:3], [[3e9, -1e9, 2e9]]])
    got = s.project(far).cpu().numpy()
    assert np.abs(got[:-1] - s.project(pts[:3]).cpu().numpy()).max() <= 1e-13 * np.abs(ref).max()


@pytest.mark.parametrize("nodes", [(3, 7), (16, 32), (18, 30)])
@pytest.mark.parametrize("count", [1, 255, 511, 512, 513, 1100])
def test_sphere_sums_counts(P, nodes, count):
    """Output counts around one and two outputs per thread, node counts that
    leave part of the last chunk: up to 540 FP64 terms of a few roundings each,
    phases of order 10 known to 1e-15: 1e-12 of the largest."""
    s, sph, (v, d) = sphere_case(P, nodes)
    rng = np.random.default_rng(5)
    dirs = directions(count, 4)
    pts = dirs * rng.uniform(1.3, 9.0, size=(count, 1))
    far = s.far_field(dirs).cpu().numpy()
    ref = sph.far_field(v, d, dirs)
    big = np.abs(sph.far_field(v, d, directions(20, 6))).max()
    assert np.abs(far - ref).max() <= 1e-12 * max(big, np.abs(ref).max())
    got = s.project(pts).cpu().numpy()
    ref = sph.project(v, d, pts * sph.k0)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


def test_sphere_sums_beyond_the_short_phase_range(P):
    """A point or vector far out sends its workgroup through the general
    sincos; its neighbours' values are the ones without it (phases of order 10,
    both routines to a unit in the last place: 1e-13 of the largest).  A point
    inside the sphere, or none at all, is refused."""
    s, sph, _ = sphere_case(P, (16, 32))
    dirs = directions(8, 4)
    a = s.project(dirs * 3.0)
    b = s.project(np.vstack([dirs * 3.0, [[0, 0, 1e12]]]))
    assert (a - b[:8]).abs().max() <= 1e-13 * a.abs().max()
    assert torch.isfinite(torch.view_as_real(b)).all()
    a = s.far_field(dirs)
    b = s.far_field(np.vstack([dirs, [[0, 1e12, 0]]]))
    assert (a - b[:8]).abs().max() <= 1e-13 * a.abs().max()
    for bad in ((0.0, 0.5, 0.0), (np.nan, 3.0, 0.0)):
        with pytest.raises(P.PstdError) as e:
            s.project(np.vstack([dirs * 3.0, [bad]]))
        assert e.value.name == "PSTD_EINVAL"
