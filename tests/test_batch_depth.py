"""Launch-model tile depth of the batched step (lbm3d_batch_plan with tz < 0,
no GPU): the workgroups of each per-XCD list take its tiles in order, each
when it is free, and no depth gives a plan whose busiest workgroup marches
more than 5% fewer planes than the depth taken, which is what the model
promises; a list with one deep tile more than workgroups counts as such."""
import heapq

import pytest

from paper_1010_4135_amd import inputs

MIXES = {
    "large and three small": [(192, 128, 128)] + [(40, 40, 40)] * 3,
    "large and one small": [(64, 64, 64), (192, 128, 128)],
    "one large": [(192, 128, 128)],
    "ragged": [(195, 140, 139), (125, 307, 111), (54, 46, 42), (12, 24, 16)],
    "headline and others": [(256, 128, 128), (128, 128, 128), (110, 69, 113), (21, 26, 15)],
    "mix": inputs.BATCH_GRIDS * 3,
    "shallow": [(300, 200, 7), (64, 64, 17)],
}


def _makespan(tiles, first, nblocks):
    last = 0
    per = nblocks // (len(first) - 1)
    for a, b in zip(first[:-1], first[1:]):
        load = [0] * per
        for t in tiles[a:b]:
            free = heapq.heappop(load) + int(t[6] - t[5]) + 3  # (3 planes before a tile's first update)
            last = max(last, free)
            heapq.heappush(load, free)
    return last


@pytest.mark.parametrize("precision", ["fp32_t64", "fp64"])
@pytest.mark.parametrize("mix", MIXES)
def test_no_depth_is_much_shorter(mix, precision):
    from paper_1010_4135_amd import lbm3d
    params = [inputs.make_params(g, (0,) * 6, precision=precision) for g in MIXES[mix]]
    chosen = _makespan(*lbm3d.lbm3d_batch_plan(params, tz=-1, cus=256))
    spans = {tz: _makespan(*lbm3d.lbm3d_batch_plan(params, tz=tz, cus=256)) for tz in (16, 32, 64, 128, 256)}
    assert chosen <= 1.05 * min(spans.values()) + 1e-9, (chosen, spans)
