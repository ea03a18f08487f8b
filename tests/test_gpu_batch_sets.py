"""Batches of several sets: pass by pass over all instances, forked onto the branches
without a graph and in graphs, against single solves."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,runs", [
    ([(160, 160, 160)] * 4, ([2] * 4, [5, 3, 4, 5])),                       # beyond the cache: 6 and 15 launches
    ([(24, 20, 32), (40, 40, 40), (48, 48, 48), (64, 64, 64)] * 7, ([3] * 28, [5] * 28)),  # 76 MB: pass by pass, forked
    ([(48, 48, 48), (64, 96, 48), (80, 80, 80), (96, 128, 160)], ([19, 17, 8, 19],)),      # 69 MB: graphs and the rest
])
def test_sets_equal_single_solves(shapes, runs):
    """The same operations in the same order on each instance, in whichever set and
    launch: psi to the bit."""
    import paper_2403_04053_amd as P
    probs = [synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=5, dft=(0, 0), theta=0.1 * i, phi=0.3)
             for i, n in enumerate(shapes)]
    states = [(synth.random_state(n, 2 * i), synth.random_state(n, 2 * i + 1)) for i, n in enumerate(shapes)]
    many = P.Batch([p for p, _ in probs])
    for i, (_, V) in enumerate(probs):
        many.set_potential(i, V)
        many.instance(i).set_state(*states[i], 0)
    for steps in runs:
        many.run(steps)
    for i, (prob, V) in enumerate(probs):
        one = P.Solver(prob)
        one.set_potential(V)
        one.set_state(*states[i], 0)
        one.run(sum(steps[i] for steps in runs))
        inst = many.instance(i)
        assert torch.equal(one.psi(), inst.psi()) and torch.equal(one.psi(1), inst.psi(1)), i
        one.close()
    many.close()
