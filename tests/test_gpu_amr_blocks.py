"""Block shapes at the edges of the refined stage's variants, against the
refined-grid oracle: leaves of 256 and of 512 threads, leaves that do not fit
LDS (the thread-per-cell variant, every ghost face filled), and a single
block along phi (a leaf is its own neighbour), with a cone CME and regrids."""
import numpy as np
import pytest

import parity
from paper_2501_15923_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,block,flux,limiter", [
    ((32, 8, 16), (8, 8, 8), 0, 0), ((32, 8, 16), (16, 8, 8), 1, 1),
    ((20, 8, 12), (10, 4, 4), 2, 1), ((24, 8, 8), (4, 4, 8), 0, 1),
    ((20, 12, 12), (10, 6, 6), 2, 0)])
def test_block_shapes_match_the_oracle(shape, block, flux, limiter):
    from oracle.amr import AmrConfig, AmrOracle
    from paper_2501_15923_amd.amr import AmrSolver
    g = synth.Grid(*shape)
    times, maps = synth.dynamic_maps(g, 3, cadence=1800.0)
    cme = np.array([[0.0, 20000.0, 5 * synth.DEG, 1.2, 40 * synth.DEG, 1.5e6, 1e-18, 0.8e6]])
    s = AmrSolver(g, block=block, max_level=2, criterion="combined", regrid_every=2,
                  max_blocks=2048, flux=flux, limiter=limiter)
    o = AmrOracle(AmrConfig(g.nr, g.nt, g.np_, g.r_in, g.r_out, g.th_min, g.th_max, br=block[0],
                            bt=block[1], bp=block[2], max_level=2, criterion="combined",
                            regrid_every=2, flux=flux, limiter=limiter))
    for x in (s, o):
        x.set_maps(times, maps)
        x.set_cmes(cme)
        x.init_radial()
    s.step(5)
    o.step(5)
    keys = s.leaves()
    assert keys == o.leaves()
    assert max(k[0] for k in keys) == 2
    a = np.stack([s.block(k) for k in keys], axis=1)
    b = np.stack([o.blocks[k].U[:, 2:-2, 2:-2, 2:-2] for k in keys], axis=1)
    e = parity.rel_errors(a[:8], b[:8])
    assert max(e.values()) <= parity.TOL_F64, e
    assert np.max(np.abs(a[8] / a[0] - b[8] / b[0])) <= parity.TOL_F64
    s.close()
