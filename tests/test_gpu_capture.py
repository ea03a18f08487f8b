"""Calls that allocate nothing once a solver has run stay capturable by a caller,
also where a longer run or more outputs would have wanted scratch memory first."""
import math

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def problem(surface, nodes=(12, 24), steps=64):
    h = 0.1
    k0 = 2 * math.pi / (8 * h)
    xy, z = (16, 19, 29, 32), (24, 27, 37, 40)
    prob = synth.Problem(n=(48, 48, 64), h=(h,) * 3, k0=k0, theta=0.5, phi=0.8, abc_cells=(4,) * 3, abc_alpha=1.0,
                         abc_U0=5.0, tfsf=(xy, xy, z), v_max=0.5 * k0 * k0 / 2, ramp_periods=0.0, n_steps=steps,
                         dft_begin=0, dft_end=steps, surf_lo=(14, 14, 22), surf_hi=(34, 34, 42))
    return prob.replace(surface_kind=1, sphere_radius=0.95, sphere_nodes=nodes) if surface == "sphere" else prob


@pytest.mark.parametrize("surface", ["box", "sphere"])
def test_captured_run_equals_an_eager_one(surface):
    """Eight steps captured after a run of one step, replayed three times with eager
    work between; the same operations in the same order: psi to the bit."""
    import paper_2403_04053_amd as P
    prob = problem(surface)
    stream = torch.cuda.Stream()
    a, b = synth.random_state(prob.n, 1), synth.random_state(prob.n, 2)
    one = P.Solver(prob, stream=stream)
    two = P.Solver(prob, stream=stream)
    for s in (one, two):
        s.set_state(a, b, 0)
        s.run(1)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        one.run(8)
    for _ in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        two.run(8)
        stream.synchronize()
    # 25 steps: the host's count of the captured solver is 9, of the same parity
    assert torch.equal(one.psi(), two.psi()) and torch.equal(one.psi(1), two.psi(1))
    for s in (one, two):
        s.close()


@pytest.mark.parametrize("count", [1, 600, 1_050_000])
def test_sphere_sums_in_one_row_of_nodes(count):
    """As many outputs as fill the chip by themselves, and captured ones, sum the
    nodes in one row: against the eager sums of a few outputs at a time, 1e-12 of
    the largest."""
    import paper_2403_04053_amd as P
    prob = problem("sphere", steps=4)
    stream = torch.cuda.Stream()
    s = P.Solver(prob, stream=stream)
    s.set_state(synth.random_state(prob.n, 1), synth.random_state(prob.n, 2), 0)
    s.run(3)
    g = np.random.default_rng(3).normal(size=(count, 3))
    dirs = torch.as_tensor(g / np.linalg.norm(g, axis=1, keepdims=True), dtype=torch.float64, device="cuda")
    few = dirs[:min(count, 500)].contiguous()
    torch.cuda.synchronize()
    if count < 1_000_000:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            far = s.far_field(dirs)
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
    else:
        far = s.far_field(dirs)
    want = s.far_field(few)
    torch.cuda.synchronize()
    assert (far[:few.shape[0]] - want).abs().max() <= 1e-12 * want.abs().max()
    s.close()
