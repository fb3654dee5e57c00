"""How calls are cut into workgroups and which kernels they take, as far as it decides precision: host logic, no GPU."""
import random

import pytest

import test_gpu_direct as direct
import test_gpu_precision as precision
import test_gpu_small_volumes as small
from gpu_util import DT, OP_POINTWISE_DGRAD, OP_POINTWISE_FWD, route
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


def test_calls_of_few_products_take_a_thread_per_output():
    """Staging bricks costs more there: 1x1x1 layers of few channels and image-like 3x3x3 ones (measured: csrc/conv_direct.hip,
    prefer_threads).  The choice is the same on every tile grid, margin width and output box growth."""
    f32, bf16 = sp3d.SP_F32, sp3d.SP_BF16
    for op, dhw, cin, cout, dt in ((OP_POINTWISE_FWD, (44, 32, 44), 40, 3, bf16), (OP_POINTWISE_FWD, (44, 32, 34), 64, 4, f32),
                                   (OP_POINTWISE_DGRAD, (128, 112, 92), 1, 4, f32), (OP_POINTWISE_FWD, (102, 110, 134), 4, 2, bf16),
                                   (sp3d.SP_OP_FWD, (84, 130, 138), 1, 3, bf16), (sp3d.SP_OP_DGRAD, (50, 36, 46), 2, 3, f32)):
        for grid, halo, grow in (((1, 1, 1), 1, 0), ((2, 2, 1), 1, 0), ((1, 2, 2), 2, 0), ((2, 1, 2), 2, 1)):
            assert route(op, sp3d.Geom(1, dhw, grid, halo, grow), cin, cout, dt)[0] == "threads", (op, dhw, grid)
    for op, dhw, cin, cout, dt in ((OP_POINTWISE_DGRAD, (90, 96, 68), 16, 128, f32), (sp3d.SP_OP_FWD, (32, 32, 32), 8, 16, f32),
                                   (sp3d.SP_OP_DGRAD, (51, 62, 70), 16, 16, f32)):
        assert route(op, sp3d.Geom(1, dhw, (1, 1, 1)), cin, cout, dt)[0] == "bricks", (op, dhw)


def test_the_direct_tests_meet_both_kernels():
    met = set()
    for n, dhw, grid, cin, cout, dtype, flat in direct.CASES:
        for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD):
            met.add((op, route(op, sp3d.Geom(n, dhw, grid, 1, 0, flat), cin, cout, DT[dtype])[0], dtype, flat))
    assert {(op, r, d) for op in (0, 1) for r in ("bricks", "threads") for d in ("f32", "bf16")} <= {m[:3] for m in met}
    assert {(r, f) for r in ("bricks", "threads") for f in (0, 1)} <= {(m[1], m[3]) for m in met}
    g = sp3d.Geom(1, (4, 6, 37), (1, 2, 1))
    for cin, cout, dtype, fwd, dgrad in ((5, 7, "f32", "threads", "threads"), (130, 600, "f32", "bricks", "bricks"),
                                         (130, 40, "bf16", "threads", "bricks"), (256, 600, "bf16", "bricks", "bricks")):
        assert route(OP_POINTWISE_FWD, g, cin, cout, DT[dtype])[0] == fwd
        assert route(OP_POINTWISE_DGRAD, g, cin, cout, DT[dtype])[0] == dgrad


@pytest.mark.parametrize("dhw, cin, cout, flat, family", [
    ((56, 88, 104), 128, 64, 0, "march"), ((64, 64, 64), 128, 128, 0, "march"), ((128, 128, 128), 128, 64, 0, "march"),
    ((4, 4, 4), 256, 256, 0, "gemm"), ((16, 16, 16), 256, 256, 0, "gemm"), ((28, 44, 52), 128, 128, 0, "gemm"),
    ((6, 48, 44), 64, 1024, 1, "march"), ((5, 240, 176), 64, 256, 1, "march"), ((16, 64, 64), 256, 256, 1, "gemm"),
    ((2, 256, 256), 128, 128, 1, "gemm"), ((2, 256, 256), 64, 64, 1, "gemm"), ((16, 256, 256), 64, 64, 1, "march")])
def test_forward_family_of_layers_measured_both_ways(dhw, cin, cout, flat, family):
    """The faster family of each (measured: csrc/conv_mfma.hip, prefer_gemm), the same on every tile grid and for every output
    box growth, so that the sums are taken in one order."""
    for grid, halo, grow in (((1, 1, 1), 1, 0), ((1, 2, 2), 1, 0), ((1, 4, 2), 2, 1), ((2, 1, 4), 1, 0)):
        if all(e % k == 0 and (e // k >= halo or (flat and i == 0)) for i, (e, k) in enumerate(zip(dhw, grid))):
            g = sp3d.Geom(1, dhw, grid, halo, grow, flat)
            assert route(sp3d.SP_OP_FWD, g, cin, cout, sp3d.SP_BF16)[0] == family, grid
            assert route(sp3d.SP_OP_DGRAD, g, cout, cin, sp3d.SP_BF16)[0] == family, grid


FWD, DGRAD, WGRAD, BF16 = sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD, sp3d.SP_OP_WGRAD, sp3d.SP_BF16


def routes(op, cases):
    return [route(op, sp3d.Geom(n, dhw, grid, 1, 0, flat), cin, cout, BF16) for n, dhw, grid, cin, cout, flat in cases]


def test_the_forward_gemm_tests_meet_the_gemm():
    """tests/test_gpu_small_volumes.py runs the implicit GEMM in every shape that it is compiled in, with and without a split."""
    met = {d[:3] + (d[3] > 1,) for op in (FWD, DGRAD) for f, d in routes(op, small.GEMM + small.NARROW_GEMM + small.SPLIT_TILES +
                                                                          small.WGRAD_GEMM) if f == "gemm"}
    assert {(c, v, b) for c in (1, 2) for v, b in ((1, 3), (1, 4), (1, 6), (2, 5), (2, 6))} <= {m[:3] for m in met}
    assert {(c, v, s) for c in (1, 2) for v in (1, 2) for s in (False, True)} <= {(m[0], m[1], m[3]) for m in met}
    for cases in (small.GEMM, small.NARROW_GEMM, small.SPLIT_TILES):
        assert all(f == "gemm" for f, _ in routes(FWD, cases))
    assert all(f == "gemm" for f, _ in routes(DGRAD, small.GEMM))
    assert all(d[1] == 2 and d[3] > 1 for _, d in routes(FWD, small.SPLIT_TILES))
    shapes = []
    for dhw, grid, ca, cb, co in small.GROWN:
        for g in (sp3d.Geom(1, dhw, grid), sp3d.Geom(1, dhw, grid, 2, 1)):
            assert route(FWD, g, ca + cb, co, BF16)[0] == "gemm"
            shapes.append((route(FWD, g, ca + cb, co, BF16)[1][1], route(DGRAD, g, ca + cb, co, BF16)[0]))
    assert {(1, "gemm"), (2, "march")} <= set(shapes)


def test_the_marching_tests_meet_the_march():
    """... and the marching kernels with one and with two chunks per launch, with and without partial sums, slices side by side."""
    fwd = routes(FWD, small.CHUNKS)
    assert all(f == "march" for f, _ in fwd)
    assert {(p, l > 1) for _, (p, _, _, l) in fwd} >= {(0, False), (1, False), (1, True)}
    assert any(d < case[1][0] // case[2][0] for case, (_, (_, _, d, _)) in zip(small.CHUNKS, fwd))
    assert {f for _, (_, f, _, _) in fwd} == {1, 2, 3}
    wgrad = routes(WGRAD, small.FINE_WGRAD)
    assert all(f in ("march", "padded") for f, _ in wgrad)
    cut = [(f, whole, d < case[1][0] // case[2][0]) for case, (f, (whole, _, d, _)) in zip(small.FINE_WGRAD, wgrad)]
    assert {whole for f, whole, fine in cut if f == "march" and fine} == {0, 1}
    assert any(f == "padded" and fine for f, _, fine in cut)
    assert {d[1] for f, d in wgrad if f == "march"} == {1, 2, 3}


def test_the_voxel_gemm_tests_meet_the_gemm():
    """... and the weight gradient as a GEMM over voxels in every shape that it is compiled in."""
    plans = routes(WGRAD, small.WGRAD_GEMM) + routes(WGRAD, [(1,) + c + (0,) for c in small.WGRAD_GATHER])
    assert all(f == "gemm" for f, _ in plans)
    assert {(t, x) for t in (2, 4) for x in (5, 6, 8)} <= {d[:2] for _, d in plans}
    assert {(t, s) for t in (2, 4) for s in (0, 1)} <= {(d[0], d[3]) for _, d in plans[:len(small.WGRAD_GEMM)]}
    assert {(t, s) for t in (2, 4) for s in (0, 1)} <= {(d[0], d[3]) for _, d in plans[len(small.WGRAD_GEMM):]}
    assert {True, False} == {d[2] > 1 for _, d in plans}


def test_the_few_channel_tests_meet_their_kernel():
    assert all(f == "few" for op in (FWD, WGRAD) for f, _ in routes(op, small.FEW + precision.FEW))
    assert {c[3] for c in small.FEW} == set(range(2, 9))


def test_the_padded_tests_meet_both_cuttings():
    """Weight gradients on zero-padded copies: the finer cutting, and the one with the fewest partial sums where only that leaves
    them room in the library's own buffer."""
    plans = {(edge, cin): route(WGRAD, sp3d.Geom(1, (edge,) * 3, (1, 1, 1)), cin, 32, BF16) for edge, cin in small.STATIC}
    assert all(f == ("padded" if cin > 8 else "few") for (_, cin), (f, _) in plans.items())
    assert {d[3] for f, d in plans.values() if f == "padded"} == {0, 1}


def flat_layers():
    layers = [(1, (16, 32, 32), (1, 1, 1), 32, 32), (1, (1, 256, 256), (1, 2, 2), 32, 32), (2, (1, 64, 64), (1, 2, 2), 32, 32),
              (1, (1, 8, 32), (1, 1, 1), 64, 64), (1, (16, 256, 256), (1, 2, 2), 64, 64)]
    rng = random.Random(21)
    for _ in range(60):
        grid = (1, rng.choice([1, 2, 4]), rng.choice([1, 2]))
        layers.append((rng.choice([1, 1, 2, 3]), (rng.randrange(1, 17), 8 * rng.randrange(1, 17) * grid[1], 32 * rng.randrange(1, 5) * grid[2]),
                       grid, 32 * rng.randrange(1, 5), 32 * rng.randrange(1, 5)))
    return layers


def test_flat_weight_gradients_have_a_step_for_every_workgroup():
    """Whole patches in 2-D are dealt out two at a time, slice by slice: no workgroup goes without (it would add a partial sum of
    zeros: 32 -> 32 on 16 x 32 x 32 had 64 workgroups for 32 steps)."""
    met = [0, 0, 0]
    for n, dhw, grid, cin, cout in flat_layers():
        family, (whole, fold, cut, groups) = route(WGRAD, sp3d.Geom(n, dhw, grid, 1, 0, 1), cin, cout, BF16)
        if family != "march":
            continue
        met[whole] += 1
        patches = n * (dhw[1] // 8) * (dhw[2] // 32)
        if whole == 2:
            assert cut == ceil(patches * dhw[0], 2)
        assert fold == 1 and 1 <= groups <= (cut if whole == 2 else patches * ceil(dhw[0], cut)), (dhw, grid, cin, cout)
    assert met[0] == 0 and met[1] >= 15 and met[2] >= 15


def test_the_flat_whole_patch_tests_meet_both_kernels():
    """Few steps per workgroup march, the others go in steps of two units (measured: csrc/wgrad_mfma.hip, launch_plan)."""
    two = [(n, dhw, grid, ca + cb, co) for n, dhw, grid, ca, cb, co in small.FLAT_PATCHES]
    for layers in (precision.FLAT, two):
        plans = [route(WGRAD, sp3d.Geom(n, dhw, grid, 1, 0, 1), cin, cout, BF16) for n, dhw, grid, cin, cout in layers]
        assert all(f == "march" for f, _ in plans) and {d[0] for _, d in plans} == {1, 2}
    for dhw, cin, cout, whole in (((1, 32, 96), 32, 32, 1), ((2, 24, 32), 32, 32, 1), ((16, 256, 256), 32, 64, 2), ((12, 512, 512), 64, 64, 2)):
        assert route(WGRAD, sp3d.Geom(1, dhw, (1, 1, 1), 1, 0, 1), cin, cout, BF16)[1][0] == whole


def test_flat_weight_gradients_of_more_pairs_than_compute_units():
    """Where a compute unit takes several channel pairs one after the other, each start has its price: few steps each are the
    GEMM's (measured: csrc/wgrad_mfma.hip, launch_plan), long ones the march's."""
    for n, dhw, cin, cout, kind in ((1, (2, 16, 32), 1024, 320, "gemm"), (1, (1, 16, 64), 768, 768, "gemm"),
                                    (1, (9, 16, 32), 1024, 1024, "gemm"), (2, (5, 16, 192), 1024, 1024, "march"),
                                    (4, (1, 96, 128), 1024, 512, "march")):
        assert route(sp3d.SP_OP_WGRAD, sp3d.Geom(n, dhw, (1, 1, 1), flat=1), cin, cout, sp3d.SP_BF16)[0] == kind, (dhw, cin, cout)


def test_the_row_tests_meet_the_rows():
    """The march of 2-D layers of up to 64 input channels goes by rows unless slices lie side by side (launch_conv_mfma)."""
    met = set()
    for case in small.ROWS:
        for op, ki in ((FWD, case[3]), (DGRAD, case[4])):
            family, (_, fold, _, _) = routes(op, [case])[0]
            rows = family == "march" and fold == 1 and ki <= 64
            assert rows or (op == DGRAD and (ki > 64 or fold > 1 or family == "gemm")), case
            if rows:
                met.add((op, ki))
    assert met == {(op, ki) for op in (FWD, DGRAD) for ki in (32, 64)}


@pytest.mark.parametrize("dhw, cin, cout, flat", [((16, 256, 256), 128, 64, 1), ((64, 64, 64), 512, 256, 0), ((64, 48, 24), 128, 128, 0)])
def test_layers_keep_the_order_of_their_sums(dhw, cin, cout, flat):
    """The family decides in which order a layer sums.  These are marched, in several launches, also where GEMM workgroups that
    stay on their compute unit have become faster (csrc/conv_mfma.hip, prefer_gemm)."""
    for grid in ((1, 1, 1), (1, 2, 2)):
        family, detail = route(FWD, sp3d.Geom(1, dhw, grid, 1, 0, flat), cin, cout, BF16)
        assert family == "march" and detail[3] > 1, grid
