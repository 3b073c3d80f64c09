"""Batched steps whose members fall into several cache-sized groups and a
tiled group, with uneven step counts: bit for bit each solve stepped alone,
across repeated runs, a change of membership, and solo steps in between."""
import numpy as np
import pytest

from paper_1010_4135_amd import inputs

pytestmark = pytest.mark.gpu

# FP32 levels: two of 126 MB pairs (a group each), one beyond the cache
# (tiled), and small ones that share the groups' room
GRIDS = [((128, 128, 64), "shock"), ((40, 24, 20), "riemann"), ((192, 128, 128), "shock"), ((128, 128, 64), "riemann"),
         ((33, 17, 9), "shock"), ((64, 64, 64), "shock"), ((16, 8, 300), "riemann")]


def _cases(precision):
    out = []
    for k, (grid, kind) in enumerate(GRIDS):
        make = inputs.shock_bubble if kind == "shock" else inputs.riemann_3d
        c = make(60 + k, grid=grid, precision=precision)
        if k % 3 == 1:
            c.params = dict(c.params, flags=8)  # velocity-major order
        out.append(c)
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp32_t64"])
def test_groups_match_solo(precision):
    from paper_1010_4135_amd import lbm3d
    cases = _cases(precision)
    rounds = [([5, 3, 2, 4, 17, 0, 6], None), ([1, 34, 1, 1, 2, 33, 3], None), ([2, 2, 0, 1, 1, 2, 2], [0, 1, 3, 4, 5, 6])]
    runs = []
    for batched in (False, True):
        solvers = []
        for c in cases:
            s = lbm3d.Solver(c.params)
            s.init(*c.fields)
            solvers.append(s)
        for steps, who in rounds:
            who = who if who is not None else list(range(len(solvers)))
            if batched:
                lbm3d.lbm3d_batch_step([solvers[k].h for k in who], [steps[k] for k in who])
            else:
                for k in who:
                    solvers[k].step(steps[k])
            for s in solvers:  # solo steps after batched ones
                s.step(1)
        runs.append([(s.get_f(), s.status()) for s in solvers])
        for s in solvers:
            s.close()
    for k, (a, b) in enumerate(zip(*runs)):
        assert a[1] == b[1], (k, GRIDS[k])
        assert np.array_equal(a[0], b[0]), (k, GRIDS[k])
