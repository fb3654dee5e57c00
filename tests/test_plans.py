"""How calls are cut into workgroups and which kernels they take, as far as it decides precision: host logic, no GPU."""
import random

import pytest

from paper_1909_03108_amd import sp3d


def ceil(a, b):
    return -(-a // b)


def coarse_groups(g, cin, cout):
    """Partial results per pair of channel blocks of the marching weight gradient, cut along D until there is an item per
    workgroup but never below 16 planes."""
    td, th, tw = g.tile
    most = max(1, 256 // ((cin // 32) * (cout // 32)))
    base = g.n * g.gd * g.gh * g.gw * ceil(th, 8) * ceil(tw, 32)
    d = td
    while base * ceil(td, d) < most and d > 16:
        d = (d + 1) // 2
    return min(base * ceil(td, d), most)


LAYERS = [((74, 38, 69), (1, 2, 1), 64, 96), ((48, 36, 36), (2, 2, 4), 32, 128), ((47, 72, 108), (1, 1, 4), 96, 32),
          ((84, 36, 36), (1, 2, 2), 192, 96), ((128, 128, 128), (4, 4, 1), 32, 32), ((99, 156, 210), (1, 2, 2), 32, 32)]
_rng = random.Random(20)
for _ in range(60):
    _grid = tuple(_rng.choice([1, 2, 4]) for _ in range(3))
    LAYERS.append((tuple(_rng.randrange(1, 60) * k for k in _grid), _grid, 32 * _rng.randrange(1, 9), 32 * _rng.randrange(1, 9)))


@pytest.mark.parametrize("dhw, grid, cin, cout", LAYERS)
def test_weight_gradient_never_sums_in_fewer_parts(dhw, grid, cin, cout):
    """Every workgroup's partial sum is one chain of fp32 additions, so that fewer of them are less exact (64 -> 96 on 74 x
    38 x 69 in 36 instead of 42: 3.7e-7 -> 4.1e-7 against 64 bits).  Cutting D finer may only add to them; the workspace says
    how many there are."""
    g = sp3d.Geom(1, dhw, grid)
    one = (27 * 32 * 32 + 32) * 4
    parts = coarse_groups(g, cin, cout) * (cin // 32) * (cout // 32)
    assert sp3d.sp_workspace_bytes(sp3d.SP_OP_WGRAD, g, cin, cout, sp3d.SP_BF16) >= parts * one
