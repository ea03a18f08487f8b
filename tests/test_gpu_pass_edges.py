"""GPU tests of the pass launches that depend on the grid's shape: the x and y
passes in one launch against the separate ones (a batch instance always takes
those), and the place of the potential term with segments along some axes."""
import numpy as np
import pytest

import synth
from oracle import pstd as opstd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available()
    import paper_2403_04053_amd as mod
    return mod


@pytest.mark.parametrize("n", [(24, 24, 20), (20, 20, 24), (40, 40, 32), (100, 100, 24), (150, 150, 20), (162, 162, 24)])
@pytest.mark.parametrize("real", [0.0, -0.5])
def test_xy_launch_equals_separate_passes(P, n, real):
    """Lengths that leave part of a tile of x rows or y columns empty, small
    tiles and large; the sums are the same operations in the same order, so
    psi and the phasors are equal to the bit."""
    prob, V = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=5, dft=(1, 4), theta=0.7, phi=0.3)
    prob = prob.replace(ramp_periods=0.1, abc_UR=real)
    a, b = synth.random_state(n, 1), synth.random_state(n, 2)
    one = P.Solver(prob)
    many = P.Batch([prob])
    inst = many.instance(0)
    for s in (one, inst):
        s.set_potential(V)
        s.set_state(a, b, 1)
    one.run(5)
    many.run(5)
    assert torch.equal(one.psi(), inst.psi()) and torch.equal(one.psi(1), inst.psi(1))
    assert torch.equal(one.phasors(), inst.phasors())


@pytest.mark.parametrize("core,halo,n", [(16, 8, (48, 32, 20)), (12, 10, (36, 24, 24)), (32, 8, (64, 96, 20)),
                                         (20, 14, (60, 40, 20)), (48, 8, (48, 96, 24)), (28, 18, (84, 56, 20))])
def test_fused_segment_blocks_equal_separate_passes(P, core, halo, n):
    """Blocks that fill the compiled pencils and ones that leave some idle, one
    block along an axis and several, with the box planes in first and last blocks;
    the sums are the same operations in the same order: equal to the bit."""
    prob, V = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=5, dft=(1, 4), theta=0.7, phi=0.3)
    prob = prob.replace(ramp_periods=0.1, sub_core=(core, core, 0), sub_halo=halo, sub_taper=3)
    a, b = synth.random_state(n, 1), synth.random_state(n, 2)
    one = P.Solver(prob)
    many = P.Batch([prob])
    inst = many.instance(0)
    for s in (one, inst):
        s.set_potential(V)
        s.set_state(a, b, 1)
    one.run(5)
    many.run(5)
    assert torch.equal(one.psi(), inst.psi()) and torch.equal(one.psi(1), inst.psi(1))
    assert torch.equal(one.phasors(), inst.phasors())


@pytest.mark.parametrize("core", [(0, 16, 16), (16, 0, 16), (16, 16, 0), (0, 0, 16), (16, 0, 0)])
def test_potential_term_with_segments_along_some_axes(P, core):
    """One step with V minus one without it is -2i dtau Gamma v psi^n at every
    cell, whichever pass takes the term: FP32 sums of a few values of order
    one, 1e-6 of the largest."""
    prob, V = synth.tiny(n=(64, 48, 64), P=4, transition=3, v0=0.5, radius_cells=5, steps=1, dft=(0, 0))
    prob = prob.replace(sub_core=core, sub_halo=8, sub_taper=3)
    a, b = (synth.random_state(prob.n, k) for k in (1, 2))
    out = []
    for pot in (V, np.zeros_like(V)):
        s = P.Solver(prob)
        s.set_potential(pot)
        s.set_state(a, b, 0)
        s.run(1)
        out.append(s.psi().cpu().numpy().astype(np.complex128))
    m = opstd.build(prob, V)
    want = -2j * m.dtau * m.Gamma * m.v * b
    assert np.abs(out[0] - out[1] - want).max() <= 1e-6 * max(np.abs(out[0]).max(), np.abs(want).max())
