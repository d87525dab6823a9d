"""GPU parity of the level pipeline (mrt_set_pipeline): four steps per launch,
one group of waves per time level, rows handed on through LDS.

Against the FP64 oracle (the stated 1e-5 on rho, u, T; 1e-12 of the
population scale in FP64) and against the one-step kernel, which rounds every
level alike (the increments are the same FMA chains; the FP64 collision's
fusion may differ per copy of the code): ragged shapes around the blocks' 120
stored columns, one row, one column, bands from one row to the whole height,
every boundary kind on every side.
"""
import numpy as np
import pytest

from helpers import field_errors, oracle_run, smooth_case
from oracle import mrt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs the GPU", allow_module_level=True)

from paper_1004_5442_amd.solver import solver_for_case  # noqa: E402

BC_SETS = [
    ("periodic", "periodic", "periodic", "periodic"),
    ("reflect", "reflect", "reflect", "reflect"),
    ("eq", "outflow", "reflect", "reflect"),
    ("reflect", "eq", "periodic", "periodic"),
    ("outflow", "reflect", "eq", "outflow"),
    ("periodic", "periodic", "reflect", "eq"),
]
# columns around one and two blocks of 120 stored columns, a wall at a block's
# first and last lanes (116..124), fewer columns or rows than the overlap
SHAPES = [((150, 37), 8), ((120, 5), 2), ((1, 7), 3), ((65, 1), 1), ((121, 12), 5), ((119, 9), 9),
          ((124, 3), 1), ((116, 40), 40), ((2, 2), 1), ((241, 4), 4), ((123, 20), 0)]


def run_pair(case, prec, rows, nsteps):
    one = solver_for_case(case, prec)
    one.set_steps_per_pass(1, 0)
    one.step(nsteps)
    pipe = solver_for_case(case, prec)
    pipe.set_pipeline(rows)
    assert pipe.pipeline() >= 1
    pipe.step(nsteps)
    a, b, fields = pipe.populations(), one.populations(), pipe.moments()
    one.close()
    pipe.close()
    return a, b, fields


@pytest.mark.parametrize("prec", ["fp64", "fp32_eq64", "fp32"])
@pytest.mark.parametrize("bc", BC_SETS)
@pytest.mark.parametrize("shape,rows", SHAPES)
def test_pipeline_matches_oracle_and_single_step(shape, rows, bc, prec):
    nx, ny = shape
    nsteps = 13                     # three passes and one single step
    case = smooth_case(nx, ny, bc, seed=3 * nx + ny)
    print(f"case {case.name} bc={bc} rows={rows} {prec} pipeline", flush=True)
    want, p = oracle_run(case, nsteps)
    got, one, fields = run_pair(case, prec, rows, nsteps)
    scale = np.abs(want).max()
    d = float(np.max(np.abs(got - one)) / scale)
    if prec == "fp64":
        err = float(np.max(np.abs(got - want)) / scale)
        assert err <= 1e-12 and d <= 1e-13, (err, d)
    else:
        err = field_errors(fields, mrt.macroscopic(want, p.b))
        assert max(err.values()) < 1e-5, err
        assert d <= (0.0 if prec == "fp32" else 1e-6), d


def test_pipeline_graphs_and_switches():
    """Graph replays, remainders of one to three steps, and switches to the
    other forms and back: the wall ghosts, which the pipeline does not write,
    are current for the step kernel that expects them."""
    case = smooth_case(300, 40, ("reflect", "eq", "reflect", "outflow"), seed=21)
    print(f"case {case.name} pipeline graphs", flush=True)
    s = solver_for_case(case, "fp32_eq64")
    total = 0
    for n, rows in ((259, 0), (1, 0), (6, 7), (3, -1), (8, 0), (1, -1)):
        s.set_pipeline(rows)
        s.step(n)
        total += n
    s.set_pipeline(0)
    s.prepare(12)
    s.step(12)
    s.set_steps_per_pass(2, 8)
    assert s.pipeline() == -1
    s.step(3)
    want, p = oracle_run(case, total + 15)
    err = field_errors(s.moments(), mrt.macroscopic(want, p.b))
    assert max(err.values()) < 1e-5, err
    s.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_eq64"])
def test_pipeline_reports_an_unhealthy_state(prec):
    from paper_1004_5442_amd.lib import UnstableError
    case = smooth_case(130, 20, BC_SETS[1], seed=2)
    s = solver_for_case(case, prec)
    s.set_pipeline(0)
    f = s.populations()
    f[:, 11, 119] = -f[:, 11, 119]          # rho < 0 in a cell of the first block's last column
    s.set_populations(f)
    s.step(4)
    with pytest.raises(UnstableError):
        s.sync()
    s.close()


def test_walls_after_a_checkpointed_run_in_the_contexts_buffers():
    """The multi-step forms leave the wall ghosts of an explicit buffer
    unwritten; the one-step kernel that expects them gets them all the same
    when that buffer is the context's own."""
    from ctypes import c_void_p

    from paper_1004_5442_amd import lib as L
    case = smooth_case(90, 30, ("reflect", "reflect", "reflect", "reflect"), seed=4)
    print(f"case {case.name} checkpointed run in the context's buffers", flush=True)
    s = solver_for_case(case, "fp32_eq64")
    s.set_pipeline(0)
    ck = s.empty_state()
    cur, other = s.buffers()
    assert L.raw().mrt_step_checkpointed(s._h, c_void_p(cur), c_void_p(other), 8, 8,
                                         (c_void_p * 1)(ck.data_ptr())) == 0
    s.set_steps_per_pass(1, 0)
    s.step(3)
    want, p = oracle_run(case, 11)
    err = field_errors(s.moments(), mrt.macroscopic(want, p.b))
    assert max(err.values()) < 1e-5, err
    s.close()


@pytest.mark.parametrize("form", ["pipeline", "tile"])
def test_walls_after_a_recorded_checkpointed_run(form):
    """A checkpointed run on the context's own buffers recorded into a graph
    of the caller's: its replays leave the wall ghosts unwritten after the
    context has refilled them, and the one-step kernel still reads those of
    the current state, after every replay."""
    from ctypes import c_void_p

    from paper_1004_5442_amd import lib as L
    case = smooth_case(90, 30, ("reflect", "reflect", "reflect", "reflect"), seed=4)
    print(f"case {case.name} {form} recorded checkpointed run", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = solver_for_case(case, "fp64", stream=st)
        if form == "pipeline":
            s.set_pipeline(0)
        ck = s.empty_state()
        cur, other = s.buffers()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            assert L.raw().mrt_step_checkpointed(s._h, c_void_p(cur), c_void_p(other), 8, 8,
                                                 (c_void_p * 1)(ck.data_ptr())) == 0
        s.set_steps_per_pass(1, 0)
        for k in (1, 2):
            graph.replay()
            s.step(2)                     # an even count: the current buffer stays the recorded one
            want, _ = oracle_run(case, 10 * k)
            got = s.populations()
            assert np.max(np.abs(got - want)) <= 1e-12 * np.abs(want).max(), k
        s.close()


def test_walls_after_fields_that_were_only_recorded():
    """Recording mrt_set_fields writes nothing yet: wall ghosts that a
    multi-step pass left stale are still renewed before the one-step kernel
    reads them."""
    case = smooth_case(90, 30, ("reflect", "reflect", "reflect", "reflect"), seed=4)
    print(f"case {case.name} recorded fields", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = solver_for_case(case, "fp64", stream=st)
        s.set_pipeline(0)
        s.step(8)
        s.set_pipeline(-1)
        fields = [torch.tensor(np.ascontiguousarray(a), device="cuda")
                  for a in (case.rho, case.ux, case.uy, case.T)]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        from ctypes import c_void_p

        from paper_1004_5442_amd import lib as L
        with torch.cuda.graph(graph, stream=st):
            assert L.raw().mrt_set_fields(s._h, *[c_void_p(t.data_ptr()) for t in fields], 1) == 0
        s.step(3)
        want, _ = oracle_run(case, 11)
        got = s.populations()
        assert np.max(np.abs(got - want)) <= 1e-12 * np.abs(want).max()
        s.close()


@pytest.mark.parametrize("form,nsteps", [("pipeline", 4), ("tile", 3)])
def test_ghost_ring_after_a_checkpointed_run_that_ends_in_the_second_buffer(form, nsteps):
    """One multi-step pass ends in f_tmp, here a buffer of the caller's whose
    ghost ring was never filled: the copy back into the context's own buffer
    leaves it with its fixed equilibria, which the pipeline then reads.  A
    checkpoint has its ring too: the one-step kernel goes on from its bytes."""
    from ctypes import c_void_p

    from paper_1004_5442_amd import lib as L
    case = smooth_case(90, 30, ("eq", "eq", "reflect", "reflect"), seed=6)
    print(f"case {case.name} {form} checkpointed run of one pass", flush=True)
    s = solver_for_case(case, "fp64")
    if form == "pipeline":
        s.set_pipeline(0)
    cur, _ = s.buffers()
    tmp, ck = s.empty_state(), [s.empty_state() for _ in range(2)]

    def run(n, segment):
        ptrs = (c_void_p * 2)(*[t.data_ptr() for t in ck])
        assert L.raw().mrt_step_checkpointed(s._h, c_void_p(cur), c_void_p(tmp.data_ptr()), segment, n, ptrs) == 0

    def check(n):
        want, _ = oracle_run(case, n)
        assert np.max(np.abs(s.populations() - want)) <= 1e-12 * np.abs(want).max(), n

    run(nsteps, nsteps)
    s.set_pipeline(0)
    s.step(4)
    check(nsteps + 4)
    s.close()
    s = solver_for_case(case, "fp64")
    if form == "pipeline":
        s.set_pipeline(0)
    cur, _ = s.buffers()
    run(2 * nsteps, nsteps)
    s.set_steps_per_pass(1, 0)
    own = next(b for b in s._bufs if b.data_ptr() == s.buffers()[0])
    own.copy_(ck[1])
    s.step(3)
    check(nsteps + 3)
    s.close()


@pytest.mark.parametrize("form", ["pipeline", "tile"])
def test_walls_of_a_state_copied_away_and_back(form):
    """A state's bytes saved after multi-step passes and brought back under
    the one-step kernel, which reads the wall ghosts among them."""
    case = smooth_case(90, 30, ("reflect", "reflect", "reflect", "reflect"), seed=8)
    print(f"case {case.name} {form} state copied away and back", flush=True)
    s = solver_for_case(case, "fp64")
    if form == "pipeline":
        s.set_pipeline(0)
    s.step(8)
    cur, _ = s.buffers()
    own = next(b for b in s._bufs if b.data_ptr() == cur)
    saved = own.clone()
    s.set_steps_per_pass(1, 0)
    s.step(2)
    own.copy_(saved)
    s.step(3)
    want, _ = oracle_run(case, 11)
    assert np.max(np.abs(s.populations() - want)) <= 1e-12 * np.abs(want).max()
    s.close()


# band heights and shapes that the launch rule gives four waves per level (248 stored columns):
# around one and two such blocks, a last block of 234 and of one column, the width of the headline grid
WIDE = [((248, 180), 1), ((241, 175), 1), ((496, 110), 1), ((730, 80), 1), ((14881, 62), 1), ((4096, 60), 4)]


@pytest.mark.parametrize("prec", ["fp32_eq64", "fp32"])
@pytest.mark.parametrize("bc", BC_SETS)
@pytest.mark.parametrize("shape,rows", WIDE)
def test_four_waves_per_level_match_single_steps(shape, rows, bc, prec):
    case = smooth_case(*shape, bc, seed=sum(shape), dt=2e-5 if max(shape) < 5000 else 5e-6)
    print(f"case {case.name} bc={bc} {prec} four waves per level", flush=True)
    one, pipe = solver_for_case(case, prec), solver_for_case(case, prec)
    one.set_steps_per_pass(1, 0)
    pipe.set_pipeline(rows)
    assert pipe.form() == ("pipeline", 4, rows, 4)
    for s in (one, pipe):
        s.step(8)
    a, b = pipe.populations(), one.populations()
    d = float(np.max(np.abs(a - b)) / np.abs(b).max())
    assert d <= (0.0 if prec == "fp32" else 1e-6), d
    one.close()
    pipe.close()


@pytest.mark.parametrize("prec,n,bc", [("fp64", 520, BC_SETS[2]), ("fp32_eq64", 720, BC_SETS[1]),
                                       ("fp32", 720, BC_SETS[4]), ("fp64", 1040, BC_SETS[0])])
def test_how_a_number_of_steps_is_split(prec, n, bc):
    """On grids that run the pipeline by default, nine steps at once (two
    passes and one left over) against nine calls: to rounding, bit for bit in
    pure FP32; bit for bit in every precision with one step per pass."""
    case = smooth_case(n, n, bc, seed=n)
    print(f"case {case.name} bc={bc} {prec} split step counts", flush=True)
    for one in (False, True):
        a, b = solver_for_case(case, prec), solver_for_case(case, prec)
        assert a.form()[0] == "pipeline"
        if one:
            for s in (a, b):
                s.set_steps_per_pass(1, 0)
        a.step(9)
        for _ in range(9):
            b.step(1)
        fa, fb = a.populations(), b.populations()
        d = float(np.max(np.abs(fa - fb)) / np.abs(fb).max())
        assert d <= (0.0 if one else {"fp64": 1e-13, "fp32_eq64": 2.4e-7, "fp32": 0.0}[prec]), d
        a.close()
        b.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_eq64"])
@pytest.mark.parametrize("bc", BC_SETS[:4])
def test_steps_left_over_after_prepared_passes(bc, prec):
    """One to three steps left over by the pipeline, launched directly, after
    prepared graphs and from either start buffer."""
    case = smooth_case(300, 40, bc, seed=31)
    print(f"case {case.name} bc={bc} {prec} left-over steps", flush=True)
    s = solver_for_case(case, prec)
    s.set_pipeline(0)
    total = 0
    for n in (6, 7, 9, 11, 14, 3):
        s.prepare(n)
        s.step(n)
        total += n
    want, p = oracle_run(case, total)
    if prec == "fp64":
        assert np.max(np.abs(s.populations() - want)) <= 1e-12 * np.abs(want).max()
    else:
        err = field_errors(s.moments(), mrt.macroscopic(want, p.b))
        assert max(err.values()) < 1e-5, err
    s.close()
