"""Grouping of the batched step (lbm3d_batch_groups, no GPU): every solve is
in one group; groups of untiled blocks fit the memory-side cache together
(192 MiB of two levels, or a member alone in up to 256); members beyond it go
tiled; a depth set by the caller tiles every member, one loaded from a tuning
cache does not."""
import ctypes

import pytest

from paper_1010_4135_amd import inputs

WALLS = (1, 1, 3, 3, 3, 3)
MIB = 1 << 20
BATCHES = {
    "small": [(32, 32, 32), (70, 19, 13), (65, 21, 17), (20, 12, 9)],
    "two groups and a large one": [(128, 128, 64), (40, 24, 20), (192, 128, 128), (128, 128, 64), (33, 17, 9)],
    "many": [(64, 64, 64)] * 20 + [(30, 50, 41)] * 7,
    "ragged": [(97, 31, 130), (255, 33, 65), (3, 200, 50), (128, 128, 128), (1, 1, 64)],
}


def _params(grids, precision):
    return [inputs.make_params(g, WALLS if min(g) > 1 else (0,) * 6, precision=precision) for g in grids]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_t64"])
@pytest.mark.parametrize("batch", BATCHES)
def test_groups_fit_the_cache(batch, precision):
    from paper_1010_4135_amd import lbm3d
    grids = BATCHES[batch]
    group, tiled = lbm3d.lbm3d_batch_groups(_params(grids, precision))
    bytes_of = [a * b * c * 30 * (8 if precision == "fp64" else 4) for a, b, c in grids]
    assert sorted(set(group)) == list(range(max(group) + 1))
    for j in set(group):
        who = [k for k in range(len(grids)) if group[k] == j]
        assert len({tiled[k] for k in who}) == 1
        if not tiled[who[0]]:
            total = sum(bytes_of[k] for k in who)
            assert total <= 192 * MIB or (len(who) == 1 and total <= 256 * MIB)
    if not all(tiled):
        assert all(tiled[k] for k in range(len(grids)) if bytes_of[k] > 256 * MIB)
    if batch == "small":
        assert not any(tiled)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_t64"])
def test_only_a_depth_set_by_the_caller_tiles_every_member(precision, tmp_path):
    from paper_1010_4135_amd import lbm3d
    ps = _params(BATCHES["small"], precision)
    try:
        lbm3d.lbm3d_batch_set_depth(precision, 16)
        assert lbm3d.lbm3d_batch_groups(ps) == ([0] * len(ps), [True] * len(ps))
        # (servers take the model's depth, and its groups)
        assert not any(lbm3d.lbm3d_batch_groups(ps, tz=-1)[1])
        if lbm3d.lbm3d_device_count() == 0:
            src = tmp_path / "tune.txt"
            src.write_text("lbm3d-tune 2 none\nbatch %d 32\n" % lbm3d.PRECISIONS[precision])
            lbm3d.lbm3d_tune_load(str(src))
            assert not any(lbm3d.lbm3d_batch_groups(ps)[1])
    finally:
        lbm3d.lbm3d_batch_set_depth(precision, 0)
    assert not any(lbm3d.lbm3d_batch_groups(ps)[1])
    assert all(lbm3d.lbm3d_batch_groups(ps, tz=16)[1])


def test_bad_arguments_are_refused():
    from paper_1010_4135_amd import lbm3d
    ps = _params(BATCHES["small"][:2], "fp32")
    mixed = [ps[0], dict(ps[1], precision="fp64")]
    for bad, cus in ((mixed, 256), ([dict(ps[0], c1=0.0)], 256), ([dict(ps[0], flags=lbm3d.UPWIND2)], 256), (ps, 0)):
        with pytest.raises(lbm3d.LbmError) as ei:
            lbm3d.lbm3d_batch_groups(bad, cus=cus)
        assert ei.value.code == lbm3d.E_INVAL
    arr = (lbm3d.lbm3d_params * 1)(lbm3d.make_params(ps[0]))
    one = (ctypes.c_int32 * 1)()
    assert lbm3d._lib.lbm3d_batch_groups(arr, 1, 0, 256, None, one) == lbm3d.E_INVAL
    assert lbm3d._lib.lbm3d_batch_groups(arr, 1, 0, 256, one, None) == lbm3d.E_INVAL
