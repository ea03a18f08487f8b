"""Box far fields captured by a caller, and what runs captured by a caller leave in
the surface sums."""
import math

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def problem(surface="box", steps=400):
    h = 0.1
    k0 = 2 * math.pi / (8 * h)
    xy, z = (16, 19, 29, 32), (24, 27, 37, 40)
    prob = synth.Problem(n=(48, 48, 64), h=(h,) * 3, k0=k0, theta=0.5, phi=0.8, abc_cells=(4,) * 3, abc_alpha=1.0,
                         abc_U0=5.0, tfsf=(xy, xy, z), v_max=0.5 * k0 * k0 / 2, ramp_periods=0.0, n_steps=steps,
                         dft_begin=0, dft_end=steps, surf_lo=(14, 14, 22), surf_hi=(34, 34, 42))
    return prob.replace(surface_kind=1, sphere_radius=0.95, sphere_nodes=(12, 24)) if surface == "sphere" else prob


def directions(count):
    g = np.random.default_rng(3).normal(size=(count, 3))
    return torch.as_tensor(g / np.linalg.norm(g, axis=1, keepdims=True), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("warm", ["directions", "points"])
def test_captured_box_far_field(warm):
    """A far field of more directions than any call before it, captured; then larger
    eager calls of both projections, which must not move what the graph uses: each
    replay is the eager result on the sums of the moment but for the incident sum
    they are divided by, which the graph took from the capture (without a ramp, the
    number of window steps): one more rounding of each phasor, 1e-14 of the largest."""
    import paper_2403_04053_amd as P
    prob = problem()
    stream = torch.cuda.Stream()
    s = P.Solver(prob, stream=stream)
    s.set_state(synth.random_state(prob.n, 1), synth.random_state(prob.n, 2), 0)
    s.run(3)
    dirs, more = directions(70001), directions(150000)
    pts = directions(4000) * 40.0
    torch.cuda.synchronize()
    if warm == "directions":
        s.far_field(dirs[:64].contiguous())
    else:
        s.project(pts[:64].contiguous())
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        far = s.far_field(dirs)
    for _ in range(3):
        s.run(5)
        s.far_field(more)
        s.project(pts)
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        want = s.far_field(dirs)
        stream.synchronize()
        assert torch.isfinite(torch.view_as_real(want)).all() and want.abs().max() > 0
        assert (far * (3 / s.step) - want).abs().max() <= 1e-14 * want.abs().max()
    s.close()


@pytest.mark.parametrize("surface", ["box", "sphere"])
def test_captured_run_leaves_the_sums_of_an_eager_one(surface):
    """Eight steps captured before the solver has run more than one, replayed between
    eager runs of four (from the first of which a box surface stages its plane values,
    while the graph goes on adding each to the sums): the same terms in the same order,
    so states and surface sums are equal to the bit, behind the saved state's header of
    80 bytes (the host counts captured steps once)."""
    import paper_2403_04053_amd as P
    prob = problem(surface)
    stream = torch.cuda.Stream()
    a, b = synth.random_state(prob.n, 1), synth.random_state(prob.n, 2)
    one, two = P.Solver(prob, stream=stream), P.Solver(prob, stream=stream)
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
        one.run(4)
        two.run(8)
        two.run(4)
        stream.synchronize()
        x, y = one.save_state(), two.save_state()
        assert torch.equal(x[80:], y[80:])
    for s in (one, two):
        s.close()
