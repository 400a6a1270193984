"""The number of phi planes a stage block marches over is chosen from the
grid's size when the caller leaves it open.  It decides only how the work is
cut: the states of a default solver, of forced chunks and of a default
ensemble are bitwise equal, from grids with less than one block per CU to
ragged ones, with chunks that do and do not divide n_phi."""
import numpy as np
import pytest

from paper_2501_15923_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 5, 3), (64, 16, 32), (97, 23, 37), (150, 30, 60),
                                   (241, 40, 67)])
@pytest.mark.parametrize("precision,limiter", [(64, 0), (32, 1), (64, 2)])
def test_default_planes_match_forced_planes(shape, precision, limiter):
    from paper_2501_15923_amd.ensemble import Ensemble
    from paper_2501_15923_amd.solver import Solver
    g = synth.Grid(*shape)
    maps = synth.relax_map(g, 5)[None]
    states = []
    for planes in (None, 1, min(7, g.np_), g.np_):
        s = Solver(g, precision=precision, limiter=limiter)
        s.set_maps(np.zeros(1), maps)
        if planes is not None:
            s.set_launch(2, 64, planes, 1)
        s.init_radial()
        s.step(5)
        states.append((s.clock()["t_code"], s.get_state(kind=1)))
        s.close()
    e = Ensemble([g, g], precision=precision, limiter=limiter)
    for r in e.runs:
        r.set_maps(np.zeros(1), maps)
        r.init_radial()
    e.step(5)
    states += [(r.clock()["t_code"], r.get_state(kind=1)) for r in e.runs]
    e.close()
    for t, u in states[1:]:
        assert t == states[0][0]
        assert np.array_equal(u, states[0][1])
