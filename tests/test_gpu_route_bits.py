"""Every compiled length on the launches it may take: a single solve (x and y passes in
one launch where the axes are alike) against a batch of one (separate passes)."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = (16,  # the least that holds absorber, taper and surface
           20, 24, 32, 40, 48, 64, 80, 96, 100, 108, 120, 128, 144, 150, 160, 162, 180, 192, 256, 288)


@pytest.mark.parametrize("N", LENGTHS)
@pytest.mark.parametrize("real", [0.0, -0.5])
def test_batch_of_one_equals_a_single_solve(N, real):
    """The same operations in the same order, so psi and the phasors are equal to the
    bit."""
    import paper_2403_04053_amd as P
    n = (N, N, 24)
    prob, _ = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=4, dft=(1, 3), theta=0.7, phi=0.3)
    prob = prob.replace(ramp_periods=0.1, abc_UR=real)
    a, b = synth.random_state(n, 1), synth.random_state(n, 2)
    one = P.Solver(prob)
    many = P.Batch([prob])
    inst = many.instance(0)
    for s in (one, inst):
        s.set_state(a, b, 0)
    one.run(4)
    many.run(4)
    assert torch.equal(one.psi(), inst.psi()) and torch.equal(one.psi(1), inst.psi(1))
    assert torch.equal(one.phasors(), inst.phasors())
    one.close()
    many.close()


@pytest.mark.parametrize("core,halo,n", [(14, 9, (28, 42, 20)), (26, 11, (52, 78, 20)), (40, 12, (80, 40, 24)),
                                         (48, 8, (48, 96, 20)), (12, 10, (36, 24, 20))])
def test_segment_blocks_fused_and_apart(core, halo, n):
    """The fused x and y passes, with pencils idle and without, against the two passes
    of one solver, set by tile shape; the same operations in the same order, so psi and
    the phasors are equal to the bit."""
    import paper_2403_04053_amd as P
    prob, V = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=9, dft=(1, 8), theta=0.7, phi=0.3)
    prob = prob.replace(ramp_periods=0.1, sub_core=(core, core, 0), sub_halo=halo, sub_taper=3)
    a, b = synth.random_state(n, 1), synth.random_state(n, 2)
    N = core + 2 * halo
    fused = {32: (4, 16), 48: (6, 32), 64: (8, 48)}[N]
    n1, _, pencils, _ = P.pstd_tile_variants(N, segmented=True)[0]
    out = []
    for shape in ((*fused, -1), (n1, pencils, 0)):
        s = P.Solver(prob)
        s.set_potential(V)
        for axis in (0, 1):
            s.set_tile(axis, *shape)
            assert s.tiles()[axis][3:] == shape[1:]
        s.set_state(a, b, 0)
        s.run(8)
        out.append((s.psi(), s.psi(1), s.phasors()))
        s.close()
    assert all(torch.equal(x, y) for x, y in zip(*out))
