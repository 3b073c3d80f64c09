"""Both kernels of the batched step, each in every precision: the tiled one
(every member of a batch whose depth was set goes by tiles) and the untiled
blocks (small members otherwise), over the same mix of plane orders, ragged
and one-column tails, fixed, extrapolating and reflecting faces.  Members are
compared bit for bit with the same solve stepped alone, which steps untiled
here, across uneven counts below and above a graph's 16 steps, solo steps
between batches (which leave the layers in memory behind, and the tiles read
some of them), poisoned buffers and the allocation-free entry point; the FP64
members also with the FP64 oracle (relative L1 1e-12 per field, the FP64
parity bound)."""
import contextlib

import numpy as np
import pytest

from paper_1010_4135_amd import inputs, metrics

pytestmark = pytest.mark.gpu

P, O, I, R = inputs.PERIODIC, inputs.OUTFLOW, inputs.INFLOW, inputs.REFLECT
VM = 8  # velocity-major order
MIX = [
    ((70, 19, 13), (O, O, R, R, O, O), 0), ((65, 21, 17), (R, O, O, R, R, O), VM), ((64, 19, 11), (P,) * 6, 0),
    ((128, 24, 16), (I, O, R, R, R, R), 0), ((129, 9, 20), (O, I, I, O, O, I), 0), ((20, 12, 9), (P,) * 6, VM),
    ((33, 17, 40), (I, I, O, I, I, R), 0), ((40, 12, 10), (O, O, P, P, P, P), VM),
]
ROUNDS = ([5, 3, 1, 4, 2, 6, 3, 0], [19, 40, 16, 23, 1, 17, 33, 18], [2, 1, 3, 17, 4, 2, 1, 5])
# tile depths that cut the members' planes, leave one over, and exceed them
KERNELS = [5, 16, 200, None]


def _lib():
    from paper_1010_4135_amd import lbm3d
    return lbm3d


@contextlib.contextmanager
def _kernel(precision, depth):
    lbm3d = _lib()
    if depth:
        lbm3d.lbm3d_batch_set_depth(precision, depth)
    try:
        yield
    finally:
        lbm3d.lbm3d_batch_set_depth(precision, 0)


def _cases(precision):
    out = []
    for k, (grid, bc, flags) in enumerate(MIX):
        c = inputs.smooth_periodic(70 + k, grid=grid, precision=precision)
        c.params = dict(c.params, bc=bc, inflow=[list(s) for s in inputs.fixed_states()], flags=flags)
        out.append(c)
    return out


def _solvers(cases):
    out = []
    for c in cases:
        s = _lib().Solver(dict(c.params))
        s.init(*c.fields)
        out.append(s)
    return out


def _bits(f):
    return f.view(np.uint64 if f.dtype == np.float64 else np.uint32)


@pytest.mark.parametrize("depth", KERNELS, ids=lambda d: "tiles%d" % d if d else "blocks")
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_t64"])
def test_members_match_solo_runs(precision, depth):
    lbm3d = _lib()
    cases = _cases(precision)
    batch, alone = _solvers(cases), _solvers(cases)
    with _kernel(precision, depth):
        tiled = lbm3d.lbm3d_batch_groups([c.params for c in cases])[1]
        assert tiled == [depth is not None] * len(cases)
        for r, steps in enumerate(ROUNDS):
            if r == 2:
                for s in batch:
                    s.poison_next()
                lbm3d.lbm3d_batch_step_noalloc([s.h for s in batch], steps)
            else:
                lbm3d.lbm3d_batch_step([s.h for s in batch], steps)
            for s, a, n in zip(batch, alone, steps):
                assert a.get_tile()[0] == 0
                s.step(3)
                a.step(n + 3)
    for k, (c, s, a) in enumerate(zip(cases, batch, alone)):
        assert s.status() == a.status(), (precision, depth, MIX[k])
        assert np.array_equal(_bits(s.get_f()), _bits(a.get_f())), (precision, depth, MIX[k])
        if precision == "fp64" and depth:
            import oracle
            o = oracle.Oracle(dict(c.params, flags=0))
            o.init(*c.fields)
            o.step(sum(r[k] for r in ROUNDS) + 9)
            assert metrics.max_rel_l1(s.moments(), o.moments()) <= 1e-12, MIX[k]
    for s in batch + alone:
        s.close()


@pytest.mark.parametrize("depth", [16, None], ids=["tiles", "blocks"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_t64"])
def test_health_of_one_member_only(precision, depth):
    """A NaN planted in one member shows in its health word and nowhere
    else."""
    lbm3d = _lib()
    cases = _cases(precision)
    batch, alone = _solvers(cases), _solvers(cases)
    for who in (batch, alone):
        f = who[2].get_f()
        f[3, 5, 7, 11] = np.nan
        who[2].set_f(f)
    steps = [2, 3, 4, 2, 3, 4, 2, 3]
    with _kernel(precision, depth):
        lbm3d.lbm3d_batch_step([s.h for s in batch], steps)
    for k, (s, a, n) in enumerate(zip(batch, alone, steps)):
        a.step(n)
        assert s.status() == a.status(), MIX[k]
        assert bool(s.status()[0] & lbm3d.HEALTH_NONFINITE) == (k == 2), MIX[k]
        x, y = s.get_f(), a.get_f()
        assert np.array_equal(np.isnan(x), np.isnan(y))
        assert np.array_equal(x[~np.isnan(x)], y[~np.isnan(y)]), MIX[k]
    for s in batch + alone:
        s.close()


@pytest.mark.parametrize("grid", [(64, 1, 40000), (8, 262200, 1)], ids=["planes40000", "rows262200"])
def test_tiled_member_with_indices_beyond_16_bits(grid):
    lbm3d = _lib()
    cases = [inputs.smooth_periodic(31, grid=grid, amp=0.2, precision="fp32"),
             inputs.smooth_periodic(32, grid=(32, 16, 8), amp=0.2, precision="fp32")]
    batch, alone = _solvers(cases), _solvers(cases)
    with _kernel("fp32", 32):
        assert all(lbm3d.lbm3d_batch_groups([c.params for c in cases])[1])
        lbm3d.lbm3d_batch_step([s.h for s in batch], [5, 3])
    for s, a, n in zip(batch, alone, (5, 3)):
        a.set_tile(0, 1)
        a.step(n)
        assert np.array_equal(s.get_f(), a.get_f())
        s.close()
        a.close()


# three groups of untiled blocks and a tiled member beyond the cache
GROUPS = {
    "fp64": [((128, 128, 64), WB) for WB in ((O, O, R, R, O, O),) * 2] + [((65, 33, 20), (R, O, O, R, R, O)),
                                                                         ((192, 128, 100), (I, O, R, R, R, R))],
    "fp32": [((128, 128, 100), (O, O, R, R, O, O)), ((128, 128, 101), (P,) * 6), ((65, 33, 20), (R, O, O, R, R, O)),
             ((192, 128, 129), (I, O, R, R, R, R))],
}
GROUPS["fp32_t64"] = GROUPS["fp32"]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_t64"])
def test_groups_of_both_kernels_in_one_run(precision):
    """Runs longer than a graph over several groups, with uneven counts, and a
    second run on the states the first one left."""
    lbm3d = _lib()
    cases = []
    for k, (grid, bc) in enumerate(GROUPS[precision]):
        c = inputs.smooth_periodic(90 + k, grid=grid, precision=precision, amp=0.1)
        c.params = dict(c.params, bc=bc, inflow=[list(s) for s in inputs.fixed_states()])
        cases.append(c)
    group, tiled = lbm3d.lbm3d_batch_groups([c.params for c in cases])
    assert tiled == [False, False, False, True] and len(set(group)) == 4, (group, tiled)
    batch, alone = _solvers(cases), _solvers(cases)
    for steps in ([21, 17, 34, 18], [3, 16, 1, 5]):
        lbm3d.lbm3d_batch_step([s.h for s in batch], steps)
        for a, n in zip(alone, steps):
            a.step(n)
    for k, (s, a) in enumerate(zip(batch, alone)):
        assert s.status() == a.status(), k
        assert np.array_equal(_bits(s.get_f()), _bits(a.get_f())), k
        s.close()
        a.close()
