"""GPU parity of the projection kernels at the edges of their launch shapes
(counts that leave part of a workgroup, wave or split idle), against the FP64
oracle on the same phasors."""
import math

import numpy as np
import pytest

import synth
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
