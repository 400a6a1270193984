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


@pytest.mark.parametrize("nt", [256, 257])  # 1024 and 1028 blocks of boundary columns
@pytest.mark.parametrize("graphs", [1, 0])
def test_step_end_of_many_columns_matches_the_oracle(nt, graphs):
    """Up to 1024 blocks of boundary columns a step ends in one launch, beyond
    that in two (clock and probes, then the next boundary): time-dependent
    maps, a CME with its tracer, logged probes and an end time on both sides
    of the line, replayed and launched directly."""
    import oracle
    import parity
    from paper_2501_15923_amd.solver import Solver
    g = synth.Grid(4, nt, 512)
    times, maps = synth.dynamic_maps(g, 3, n_maps=3, cadence=100.0)
    cme = np.array([[0.0, 7200.0, 5 * synth.DEG, 1.2, 30 * synth.DEG, 1.2e6, 1e-18, 0.8e6]])
    s = Solver(g, tracer=True, probe_log_rows=16)
    o = oracle.Oracle(g.nr, g.nt, g.np_, tracer=True)
    s.set_launch(2, 64, 0, graphs)
    s.set_probes(synth.probe_tables(synth.DAY, 1), cadence=0.0)
    for x in (s, o):
        x.set_maps(times, maps)
        x.set_cmes(cme)
        x.init_radial()
    t_end = s.clock()["next_dt"] * 6.5
    print("columns", g.nt * g.np_, "graphs", graphs, flush=True)
    a, b = s.step(12, t_end=t_end), o.step(12, t_end=t_end)
    assert a["steps"] == b["steps"] and 4 < a["steps"] < 12
    assert s.clock()["t"] == pytest.approx(t_end, rel=1e-15)
    parity.assert_parity(s.get_state(kind=1), o.get_state(kind=oracle.CONS_CODE))
    assert np.max(np.abs(s.get_tracer() - o.get_tracer())) <= parity.TOL_F64
    log, n = s.read_probe_log(16)
    assert n == a["steps"]
    assert np.allclose(log[-1], s.sample_probes(), rtol=1e-12, atol=0.0, equal_nan=True)
    s.close()


@pytest.mark.parametrize("nt", [256, 257])
def test_profiled_steps_are_the_launches_of_a_step(nt):
    """Timed steps launch what a step launches: the boundary has a time of its
    own only where it has a launch of its own; state and clock bitwise."""
    from paper_2501_15923_amd.solver import Solver
    g = synth.Grid(4, nt, 512)
    maps = synth.relax_map(g, 7)[None]
    states = []
    for profiled in (False, True):
        s = Solver(g)
        s.set_maps(np.zeros(1), maps)
        s.init_radial()
        print("columns", g.nt * g.np_, "profiled", profiled, flush=True)
        if profiled:
            ms = s.profile_steps(3)
            assert (ms[0] == 0.0) == (nt == 256)
            assert np.all(ms[1:] > 0.0)
        else:
            s.step(3)
        states.append((s.clock(), s.get_state(kind=1)))
        s.close()
    assert states[0][0] == states[1][0]
    assert np.array_equal(states[0][1], states[1][1])


def test_the_launch_shape_reported_is_the_one_run():
    """What a benchmark states as its launch shape: the count chosen by the
    rule where none was set, else the one set; one plane a block for the
    thread-per-cell variant."""
    from paper_2501_15923_amd.solver import Solver
    s = Solver(synth.Grid(600, 60, 120))
    assert s.launch() == (2, 64, 12)
    s.set_launch(2, 32, 15, 1)
    assert s.launch() == (2, 32, 15)
    s.set_launch(0, 0, 0, 1)
    assert s.launch() == (2, 64, 12)
    s.set_launch(1, 128, 8, 1)
    assert s.launch() == (1, 128, 1)
    s.close()
    s = Solver(synth.Grid(9, 5, 3))
    variant, tile_r, planes = s.launch()
    assert (variant, tile_r) == (2, 64) and 1 <= planes <= 3
    s.close()


@pytest.mark.parametrize("shape", [(1, 4, 6), (64, 32, 32), (97, 23, 37)])
@pytest.mark.parametrize("precision", [64, 32])
def test_state_from_the_host_and_from_the_device(shape, precision):
    """A state put in by chunks from the host (one, exactly one and two of
    65536 cells) and as a whole from the device: the same state and first dt
    bitwise, the dt of its fastest cell."""
    import torch
    from paper_2501_15923_amd.solver import Solver
    g = synth.Grid(*shape)
    maps = synth.relax_map(g, 3)[None]
    src = Solver(g, precision=precision)
    src.set_maps(np.zeros(1), maps)
    src.init_radial()
    dt = src.clock()["next_dt"]
    u = src.get_state(kind=1)
    src.close()
    out = []
    for state in (u, torch.from_numpy(u).cuda()):
        s = Solver(g, precision=precision)
        s.set_maps(np.zeros(1), maps)
        s.set_state(state, kind=1)
        out.append((s.clock()["next_dt"], s.get_state(kind=1)))
        s.close()
    for next_dt, v in out:
        assert next_dt == dt
        assert np.array_equal(v, u)
