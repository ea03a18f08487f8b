"""GPU tests of the pass launches that depend on the grid's shape: the place of
the potential term with segments along some axes."""
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
