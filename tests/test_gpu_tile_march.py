"""GPU parity of the tile march, the default of small grids: several steps per
launch, one wave per row of a tile, boundaries by shadow cells and by the wall
cells themselves.

Against the oracle (1e-12 of the population scale in FP64, the stated 1e-5 on
the fields in FP32 storage) and against the one-step kernel (FP32 bit for bit:
the same FMA chains; two FP32 ulps with FP64 collision, 1e-13 in FP64, whose
fusion may differ per copy of the code), and n steps in one call against n
calls bit for bit.  Shapes around the tiles (64 columns and 8, 12 or 16 rows
less the overlap), one row, one column, grids smaller than the overlap.
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
SHAPES = [(1, 7), (65, 1), (2, 2), (1, 1), (56, 8), (57, 9), (113, 17), (128, 96), (3, 40)]


@pytest.mark.parametrize("prec", ["fp64", "fp32_eq64", "fp32"])
@pytest.mark.parametrize("bc", BC_SETS)
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_march_matches_oracle_and_single_steps(shape, bc, prec):
    nx, ny = shape
    nsteps = 13
    case = smooth_case(nx, ny, bc, seed=5 * nx + ny)
    print(f"case {case.name} bc={bc} {prec} default launch", flush=True)
    want, p = oracle_run(case, nsteps)
    one = solver_for_case(case, prec)
    one.set_steps_per_pass(1, 0)
    one.step(nsteps)
    tile = solver_for_case(case, prec)
    tile.step(nsteps)
    again = solver_for_case(case, prec)
    for n in (1, 5, 7):
        again.step(n)
    got, ref, scale = tile.populations(), one.populations(), np.abs(want).max()
    assert np.array_equal(again.populations(), got)
    d = float(np.max(np.abs(got - ref)) / scale)
    assert d <= {"fp64": 1e-13, "fp32_eq64": 2.4e-7, "fp32": 0.0}[prec], d
    if prec == "fp64":
        assert float(np.max(np.abs(got - want)) / scale) <= 1e-12
    else:
        err = field_errors(tile.moments(), mrt.macroscopic(want, p.b))
        assert max(err.values()) < 1e-5, err
    for s in (one, tile, again):
        s.close()
