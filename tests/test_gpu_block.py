"""The untiled step kernel at the sizes where its 32 x 8 blocks can go wrong:
exactly covered, one node short or over, pairs of face nodes split between
blocks or wavefronts, single nodes per axis, every boundary kind, both plane
orders.  Against the FP64 oracle (relative L1 1e-12 per field, the FP64
parity bound), and in every precision bit for bit against the tiled kernel,
which evaluates the same operations per node."""
import numpy as np
import pytest

from paper_1010_4135_amd import inputs, metrics

pytestmark = pytest.mark.gpu

P, O, I, R = inputs.PERIODIC, inputs.OUTFLOW, inputs.INFLOW, inputs.REFLECT
CASES = [
    ((32, 8, 4), (P,) * 6), ((33, 9, 3), (P,) * 6), ((1, 1, 1), (P,) * 6), ((2, 3, 2), (P,) * 6),
    ((64, 16, 5), (O, O, O, O, O, O)), ((33, 9, 5), (O, O, O, O, O, O)), ((34, 10, 2), (O, O, O, O, O, O)),
    ((65, 17, 3), (R, R, R, R, R, R)), ((32, 8, 2), (R, O, O, R, R, O)), ((2, 2, 2), (O, R, R, O, O, R)),
    ((3, 3, 3), (R, O, O, R, R, O)), ((31, 7, 4), (I, O, R, R, R, R)), ((64, 9, 4), (I, O, R, R, R, R)),
    ((33, 11, 6), (O, I, I, O, O, I)), ((128, 10, 4), (I, I, I, I, I, I)), ((40, 12, 4), (I, I, O, I, I, R)),
]


def _case(grid, bc, precision, flags=0):
    c = inputs.smooth_periodic(41, grid=grid, precision=precision)
    c.params = dict(c.params, bc=bc, inflow=[list(s) for s in inputs.fixed_states()], flags=flags)
    return c


def _run(c, tile, steps=5):
    from paper_1010_4135_amd import lbm3d
    with lbm3d.Solver(c.params) as s:
        s.set_tile(*tile)
        s.init(*c.fields)
        s.step(steps)
        return s.get_f(), s.moments()


@pytest.mark.parametrize("vm", [0, 8], ids=["plane_major", "velocity_major"])
@pytest.mark.parametrize("k", range(len(CASES)))
def test_block_edges(k, vm):
    import oracle
    grid, bc = CASES[k]
    for precision in ("fp64", "fp32", "fp32_t64"):
        c = _case(grid, bc, precision, vm)
        f, m = _run(c, (0, 1))
        ft, _ = _run(c, (4, 3))
        assert np.array_equal(f, ft), (grid, bc, precision)
        if precision == "fp64":
            o = oracle.Oracle(dict(c.params, flags=0))
            o.init(*c.fields)
            o.step(5)
            assert metrics.max_rel_l1(m, o.moments()) <= 1e-12, (grid, bc)


@pytest.mark.parametrize("k", [1, 5, 7, 11, 13])
def test_upwind_block_edges(k):
    import oracle
    grid, bc = CASES[k]
    c = _case(grid, bc, "fp64", 2)
    _, m = _run(c, (0, 1))
    o = oracle.Oracle(dict(c.params))
    o.init(*c.fields)
    o.step(5)
    assert metrics.max_rel_l1(m, o.moments()) <= 1e-12, (grid, bc)


def test_untiled_and_batched_steps_alternate():
    """Untiled steps leave the layers in memory behind; batched steps, which
    read some of them, give the same bits as stepping untiled throughout."""
    from paper_1010_4135_amd import lbm3d
    cases = [_case(g, b, "fp32_t64") for g, b in (CASES[5], CASES[7], CASES[11], CASES[15])]
    runs = []
    for batched in (False, True):
        solvers = []
        for c in cases:
            s = lbm3d.Solver(c.params)
            s.set_tile(0, 1)
            s.init(*c.fields)
            solvers.append(s)
        for n in (3, 2, 35):
            for s in solvers:
                s.step(n)
            if batched:
                lbm3d.lbm3d_batch_step([s.h for s in solvers], [2] * len(solvers))
            else:
                for s in solvers:
                    s.step(2)
        runs.append([s.get_f() for s in solvers])
        for s in solvers:
            s.close()
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
