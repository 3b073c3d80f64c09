"""Which kernel an untuned solve starts with on a 256-CU device, by the launch
model, and that the default gives the bits of the other kernel."""
import glob

import numpy as np
import pytest

from paper_1010_4135_amd import inputs

pytestmark = pytest.mark.gpu

P, O, R = inputs.PERIODIC, inputs.OUTFLOW, inputs.REFLECT
UNTILED = [((150, 100, 70), "fp32"), ((100, 61, 50), "fp64"), ((65, 40, 7), "fp32"), ((192, 128, 53), "fp32_t64"),
           ((130, 61, 97), "fp64")]
# (chunks of 17, 25, 40, 50 and 100 planes)
TILED = [((250, 120, 33), "fp64"), ((170, 150, 100), "fp32"), ((160, 160, 160), "fp32"), ((200, 200, 100), "fp32_t64"), ((300, 150, 100), "fp64")]


def _compute_units():
    """Of the first GPU in the KFD topology (four SIMDs each; 0: unknown)."""
    for f in sorted(glob.glob("/sys/class/kfd/kfd/topology/nodes/*/properties")):
        try:
            with open(f) as lines:
                simds = [int(line.split()[1]) for line in lines if line.startswith("simd_count")]
        except OSError:
            continue
        if simds and simds[0] > 0:
            return simds[0] // 4
    return 0


@pytest.mark.parametrize("bc", [(P,) * 6, (O, O, R, R, O, R)], ids=["periodic", "walls"])
def test_default_kernel(bc):
    if _compute_units() != 256:
        pytest.skip("the expected kernels are those of a 256-CU device")
    from paper_1010_4135_amd import lbm3d
    for want, cases in ((False, UNTILED), (True, TILED)):
        for grid, precision in cases:
            with lbm3d.Solver(inputs.make_params(grid, bc, precision=precision)) as s:
                assert (s.get_tile()[0] != 0) == want, (grid, precision, s.get_tile())


@pytest.mark.parametrize("bc", [(P,) * 6, (O, O, R, R, O, R)], ids=["periodic", "walls"])
@pytest.mark.parametrize("grid,precision", UNTILED + TILED, ids=lambda v: str(v).replace(" ", ""))
def test_default_matches_the_other_kernel(grid, precision, bc):
    from paper_1010_4135_amd import lbm3d
    c = inputs.smooth_periodic(53, grid=grid, precision=precision)
    c.params = dict(c.params, bc=bc)
    states = []
    for other in (False, True):
        with lbm3d.Solver(c.params) as s:
            if other:
                s.set_tile(*((0, 1) if s.get_tile()[0] else (4, 9)))
            s.init(*c.fields)
            s.step(3)
            states.append(s.get_f())
    assert np.array_equal(states[0], states[1])
