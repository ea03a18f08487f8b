"""The FDTD kernel's tilings against the FP64 oracle: runs of planes from the
shortest to the longest with and without a remainder, tiles of 8 and 16 rows,
cells cut off in x and y, and fields beyond the Infinity Cache."""
import numpy as np
import pytest

import synth
from oracle import fdtd as ofdtd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# runs of 3, remainders 0 to 2; 5 and 10; 16 in tiles of 8 rows; in tiles of
# 16 rows, the last one whole or cut; the same with non-temporal loads
GRIDS = [(24, 24, 24), (34, 30, 28), (62, 66, 26), (64, 96, 200), (98, 134, 150), (160, 168, 150), (160, 160, 160),
         (158, 170, 152), (288, 256, 184)]


@pytest.mark.parametrize("n", GRIDS)
def test_fdtd_tiles_match_oracle(n):
    """One step from a random state, within 1e-5 of the largest value as for
    every single FP32 step."""
    import paper_2403_04053_amd as P
    prob, V = synth.tiny(n=n, P=4, transition=2, v0=0.5, radius_cells=3, steps=50, theta=0.6, phi=2.0, dft=(0, 0))
    prob, V = prob.replace(scheme=1, ramp_periods=0.5), V.astype(np.float32).astype(np.float64)
    print(f"FDTD tiles {n}", flush=True)
    s = P.Solver(prob)
    s.set_potential(V)
    prev = synth.random_state(n, 11).astype(np.complex64)
    cur = synth.random_state(n, 12).astype(np.complex64)
    s.set_state(prev, cur, 37)
    s.run(1)
    got = s.psi(0).cpu().numpy()
    ref = ofdtd.step(ofdtd.build(prob, V), prev.astype(np.complex128), cur.astype(np.complex128), 37)
    assert np.abs(got - ref).max() < 1e-5 * np.abs(ref).max()
    s.close()
