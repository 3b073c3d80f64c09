"""Default launch shapes that are not powers of two planes deep, or are
untiled, or store plainly, by the launch model: each evaluates the same
operations per node, so a few steps give the bits of the untiled kernel."""
import numpy as np
import pytest

from paper_1010_4135_amd import inputs

pytestmark = pytest.mark.gpu

P, O, R = inputs.PERIODIC, inputs.OUTFLOW, inputs.REFLECT
CASES = [
    ((192, 128, 53), inputs.FP32), ((192, 128, 53), inputs.FP32_T64), ((250, 120, 33), inputs.FP64),
    ((150, 100, 70), inputs.FP32), ((170, 150, 100), inputs.FP32), ((130, 61, 97), inputs.FP64),
    ((100, 61, 50), inputs.FP64), ((65, 40, 7), inputs.FP32),
]


@pytest.mark.parametrize("bc", [(P,) * 6, (O, O, R, R, O, R)], ids=["periodic", "walls"])
@pytest.mark.parametrize("grid,precision", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_default_shape_matches_untiled(grid, precision, bc):
    from paper_1010_4135_amd import lbm3d
    c = inputs.smooth_periodic(47, grid=grid, precision=precision)
    c.params = dict(c.params, bc=bc)
    states = []
    for tile in (None, (0, 1)):
        with lbm3d.Solver(c.params) as s:
            if tile:
                s.set_tile(*tile)
            s.init(*c.fields)
            s.step(3)
            states.append(s.get_f())
    assert np.array_equal(states[0], states[1])
