"""Misfit gradients of one solver whose step graphs and last segment's states
are kept: repeated calls and a second potential against solvers of their own."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,steps,n_ck", [((20, 20, 24), 34, 1), ((20, 24, 20), 34, 2), ((20, 20, 24), 33, 2),
                                          ((20, 20, 24), 45, 3), ((20, 20, 24), 48, 3), ((20, 20, 24), 35, 35),
                                          ((20, 20, 24), 37, 5)])
def test_kept_graphs_and_states_change_nothing(n, steps, n_ck):
    """Segments one below, at and one above a graph's 16 steps, a shorter last
    one, one of a single step: the same operations, so equal to the bit."""
    import paper_2403_04053_amd as P
    prob, V = synth.tiny(n=n, P=3, transition=3, v0=1.0, radius_cells=2, steps=steps, dft=(5, steps))
    prob = prob.replace(ramp_periods=0.3)
    pts = np.array([[0.3, -0.2, 1.5], [-0.4, 0.1, 1.6], [0.0, 0.0, -1.7]])
    target = np.array([1.0, 0.9, 1.1])

    def gradient(s, v):
        s.set_potential(v)
        J = s.misfit(steps, pts, target, n_checkpoints=n_ck)
        return J, s.misfit_gradient().clone(), s.misfit_gradient().clone(), s.psi().clone()

    one = P.Solver(prob)
    got = [gradient(one, v) for v in (V, 0.5 * V, V)]
    want = []
    for v in (V, 0.5 * V):
        s = P.Solver(prob)
        want.append(gradient(s, v))
        s.close()
    for g, w in zip(got, (want[0], want[1], want[0])):
        assert g[0] == w[0] and all(torch.equal(a, b) for a, b in zip(g[1:], w[1:]))
        assert torch.equal(g[1], g[2]) and float(g[1].abs().max()) > 0
    one.close()
