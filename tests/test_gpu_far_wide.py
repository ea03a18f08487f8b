"""Box far fields of vectors beyond unit length (the formula holds for any vector):
their blocks of 16 directions, and what they cost."""
import time

import numpy as np
import pytest

import synth
from oracle import ntdf as ontdf
from oracle import pstd as opstd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def case(n):
    import paper_2403_04053_amd as P
    prob, _ = synth.tiny(n=n, P=3, transition=2, v0=0.5, radius_cells=3, steps=1, dft=(0, 1))
    prob = prob.replace(ramp_periods=0.0, theta=0.6, phi=0.9)
    s = P.Solver(prob)
    s.set_state(synth.random_state(n, 1), synth.random_state(n, 2), 0)
    s.run(1)
    return prob, s


def vectors(count, lo, hi, seed=0):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(count, 3))
    return d / np.abs(d).max(1, keepdims=True) * rng.uniform(lo, hi, size=(count, 1))


@pytest.mark.parametrize("n", [(24, 20, 32), (40, 150, 20), (16, 24, 108)])
@pytest.mark.parametrize("count,every", [(1, 1), (17, 1), (300, 1), (4100, 1), (300, 47), (5000, 1111)])
def test_vectors_beyond_unit_length(n, count, every):
    """Lengths that leave part of the tiles of 4 and 16 empty; blocks all of such
    vectors, and ones with a single one among unit vectors, whose values stay those of
    the series.  Sums of some hundred FP64 terms with phases of up to 3 half widths:
    1e-12 of the largest."""
    prob, s = case(n)
    phi, dphi = s.split_phasors(s.phasors().cpu().numpy())
    box = ontdf.Box(prob.n, opstd.dxbar(prob), prob.surf_lo, prob.surf_hi)
    d = vectors(count, 0.3, 0.5)
    d[::every] = vectors(count, 1.0000001, 3.0, 1)[::every]
    got = s.far_field(d).cpu().numpy()
    some = np.unique(np.concatenate([np.arange(0, count, every)[:40], np.arange(count)[-20:]]))
    ref = ontdf.far_field(box, phi, dphi, d[some]) / prob.k0
    assert np.abs(got[some] - ref).max() <= 1e-12 * np.abs(ref).max()
    plain = np.ones(count, bool)
    plain[::every] = False
    if plain.any():
        d[::every] = 0.1
        assert np.array_equal(got[plain], s.far_field(d).cpu().numpy()[plain])
    s.close()


def test_vectors_beyond_unit_length_cost():
    """All of 8192 vectors beyond unit length, against unit ones: about 64 / 8 as many
    products per direction on the same units, so 40 times is a wide margin (a workgroup
    per direction took 200 times)."""
    _, s = case((64, 64, 64))
    took = []
    for d in (vectors(8192, 0.3, 0.5), vectors(8192, 1.5, 2.5)):
        d = torch.as_tensor(d, dtype=torch.float64, device="cuda")
        s.far_field(d)
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.far_field(d)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
    print(f"8192 directions: {took[0] * 1e6:.0f} us, beyond unit length {took[1] * 1e6:.0f} us", flush=True)
    s.close()
    assert took[1] <= 40 * took[0]
