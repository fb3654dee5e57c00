"""The convolution kernels for any channel count in fp32 arithmetic (conv_direct.hip) where their cutting can go wrong:
channel counts on both sides of a quad, of a 16-channel block and of a chunk, bricks that stick out of their tile, one
voxel per tile, every number of voxel segments per wave (it grows with voxels x output blocks), several bricks per
workgroup with and without a second channel chunk, extent-1 kernels, the 2-D variant and a grown output box.
Bounds: exact fp32 products, sums of at most 27 * 40 terms (forward, data gradient) or 30 000 voxels (weight gradient):
K 2^-24 relative to the sum of magnitudes in the worst case, sqrt(K) 2^-24 < 1e-5 of the result's rms for random
signs; bf16 tensors add one rounding of the result (1e-2 bounds one ulp, weight gradients stay fp32)."""
import numpy as np
import pytest
import torch

from oracle import conv3d, flat as flat_oracle
from paper_1909_03108_amd import sp3d, synth
from gpu_util import DT, TOL, f64, rel_err, route, to_dev, widen

pytestmark = pytest.mark.gpu

CASES = [  # n, dhw, grid, cin, cout, dtype, flat
    (1, (1, 1, 1), (1, 1, 1), 1, 1, "f32", 0),
    (1, (3, 5, 7), (1, 1, 1), 2, 3, "f32", 0),
    (2, (4, 6, 34), (2, 3, 2), 4, 4, "f32", 0),
    (1, (5, 9, 11), (1, 1, 1), 5, 15, "f32", 0),
    (1, (6, 10, 14), (1, 2, 2), 15, 16, "f32", 0),
    (1, (6, 10, 14), (2, 1, 1), 16, 17, "f32", 0),
    (1, (7, 6, 9), (1, 1, 1), 17, 33, "f32", 0),
    (1, (6, 7, 9), (1, 1, 1), 40, 12, "f32", 0),       # three chunks of input channels
    (1, (3, 4, 300), (1, 1, 1), 8, 8, "f32", 0),        # rows longer than a brick
    (1, (31, 29, 37), (1, 1, 1), 4, 16, "f32", 0),      # two voxel segments per wave (data gradient: one)
    (1, (24, 32, 34), (1, 2, 1), 6, 80, "f32", 0),      # four segments; several bricks per workgroup
    (1, (20, 20, 21), (1, 1, 1), 20, 70, "f32", 0),     # ... with two chunks
    (1, (5, 12, 18), (1, 2, 2), 16, 48, "bf16", 0),
    (1, (4, 9, 13), (1, 1, 1), 6, 10, "bf16", 0),
    (1, (5, 12, 18), (1, 2, 3), 8, 20, "f32", 1),
    (1, (3, 7, 50), (1, 1, 1), 17, 5, "bf16", 1),
    (1, (9, 14, 30), (1, 2, 2), 1, 3, "bf16", 0),       # a thread per output
    (2, (5, 8, 12), (1, 2, 2), 2, 2, "f32", 0),
    (1, (4, 20, 30), (1, 2, 2), 3, 2, "bf16", 1),
    (1, (7, 30, 22), (1, 2, 1), 6, 5, "f32", 1),
    (1, (40, 34, 36), (1, 2, 2), 1, 4, "f32", 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d-%dto%d-%s%s" % (c[1] + c[3:6] + ("-2d" if c[6] else "",)))
def test_three_passes_against_the_oracle(case):
    n, dhw, grid, cin, cout, dtype, flat = case
    dt, tol = DT[dtype], TOL[dtype]
    g = sp3d.Geom(n, dhw, grid, 1, 0, flat)
    seed = 4100 + 10 * CASES.index(case)
    x = synth.normal_volume((n,) + dhw + (cin,), seed, dtype)
    dz = synth.normal_volume((n,) + dhw + (cout,), seed + 1, dtype)
    w = synth.weights(cin, cout, seed + 2, dtype, taps=(3, 3) if flat else (3, 3, 3))
    bias = np.linspace(-0.5, 0.5, cout).astype(np.float32)
    ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, cin, cout, dt) for op in (0, 1, 2)))

    def padded(v, c):
        P = sp3d.alloc_padded(g, c, dt)
        sp3d.sp_partition(to_dev(v), P, g, c, dt)
        sp3d.sp_halo_exchange(P, g, c, dt)
        return P

    def volume(P, c):
        V = torch.empty((n,) + dhw + (c,), dtype=P.dtype, device="cuda")
        sp3d.sp_unpartition(P, V, g, c, dt)
        return f64(V)

    Px, Pz, wd = padded(x, cin), padded(dz, cout), to_dev(w)
    Py, Pdx, Pdm = (sp3d.alloc_padded(g, c, dt) for c in (cout, cin, cin))
    sp3d.conv3d_fwd(Px, wd, torch.from_numpy(bias).cuda(), Py, g, cin, cout, dt, sp3d.SP_FLAG_RELU, ws)
    sp3d.conv3d_dgrad(Pz, wd, Pdx, g, cin, cout, dt, ws)
    sp3d.conv3d_dgrad_relu(Pz, wd, Px, Pdm, g, cin, cout, dt, ws)
    dw = torch.full(tuple(w.shape), 9.0, device="cuda")
    db = torch.full((cout,), 9.0, device="cuda")
    sp3d.conv3d_wgrad(Px, Pz, dw, db, g, cin, cout, dt, ws)
    again = torch.empty_like(dw)
    sp3d.conv3d_wgrad(Px, Pz, again, None, g, cin, cout, dt, ws)
    assert torch.equal(dw, again)                       # no bias gradient asked for, and reproducible
    xv, zv, wv, bv = widen(x), widen(dz), widen(w), bias.astype(np.float64)
    O = flat_oracle if flat else conv3d
    y, dx, rw, rb = ((O.conv_fwd(xv, wv, bv, True), O.conv_dgrad(zv, wv), O.conv_wgrad(xv, zv), O.bias_grad(zv)) if flat else
                     (O.conv3d_fwd(x, wv, bv, True), O.conv3d_dgrad(dz, wv), O.conv3d_wgrad(x, dz), O.bias_grad(dz)))
    assert rel_err(volume(Py, cout), y) <= tol
    assert rel_err(volume(Pdx, cin), dx) <= tol
    assert np.array_equal(volume(Pdm, cin), np.where(xv > 0, volume(Pdx, cin), 0.0))
    assert rel_err(f64(dw), rw) <= 1e-5 and rel_err(f64(db), rb) <= 1e-5


def test_grown_box_and_wide_margin_equal_the_exchange():
    """fp32, halo 2: a layer that also computes the voxel around its tiles gives there, bit for bit, what the
    neighbour computes for itself, and nothing beyond the volume."""
    n, dhw, grid, cin, cout = 1, (10, 12, 22), (2, 2, 2), 9, 18
    x, w = synth.normal_volume((n,) + dhw + (cin,), 77, "f32"), to_dev(synth.weights(cin, cout, 78, "f32"))
    g = sp3d.Geom(n, dhw, grid, 2)
    Px = sp3d.alloc_padded(g, cin, sp3d.SP_F32)
    sp3d.sp_partition(to_dev(x), Px, g, cin, sp3d.SP_F32)
    sp3d.sp_halo_exchange(Px, g, cin, sp3d.SP_F32)
    out = []
    for grow in (0, 1):
        P = sp3d.alloc_padded(g, cout, sp3d.SP_F32)
        sp3d.conv3d_fwd(Px, w, None, P, g.grown(grow), cin, cout, sp3d.SP_F32)
        out.append(P)
    narrow = sp3d.Geom(n, dhw, grid, 1)
    ref = sp3d.alloc_padded(narrow, cout, sp3d.SP_F32)
    V = torch.empty((n,) + dhw + (cout,), device="cuda")
    sp3d.sp_unpartition(out[0], V, g, cout, sp3d.SP_F32)
    sp3d.sp_partition(V, ref, narrow, cout, sp3d.SP_F32)
    sp3d.sp_halo_exchange(ref, narrow, cout, sp3d.SP_F32)
    inner = (slice(None),) * 4 + (slice(1, -1),) * 3
    assert torch.equal(out[1][inner], ref)


def test_grown_box_of_a_thread_per_output_equals_the_exchange():
    """The same with a thread per output, on a grid whose tiles have neighbours on one side, on both and on none."""
    n, dhw, grid, cin, cout, dt = 2, (9, 8, 15), (3, 1, 3), 1, 3, sp3d.SP_F32
    x, w = to_dev(synth.normal_volume((n,) + dhw + (cin,), 79, "f32")), to_dev(synth.weights(cin, cout, 80, "f32"))
    out = []
    for halo, grow in ((1, 0), (2, 0), (2, 1)):
        g = sp3d.Geom(n, dhw, grid, halo, grow)
        Px, Py = sp3d.alloc_padded(g, cin, dt), sp3d.alloc_padded(g, cout, dt)
        assert route(sp3d.SP_OP_FWD, g, cin, cout, dt)[0] == "threads"
        sp3d.sp_partition(x, Px, g, cin, dt)
        sp3d.sp_halo_exchange(Px, g, cin, dt)
        sp3d.conv3d_fwd(Px, w, None, Py, g, cin, cout, dt)
        if not grow:
            V = torch.empty((n,) + dhw + (cout,), device="cuda")
            sp3d.sp_unpartition(Py, V, g, cout, dt)
        out.append(Py if grow else V)
    narrow = sp3d.Geom(n, dhw, grid)
    ref = sp3d.alloc_padded(narrow, cout, dt)
    sp3d.sp_partition(out[0], ref, narrow, cout, dt)
    sp3d.sp_halo_exchange(ref, narrow, cout, dt)
    inner = (slice(None),) * 4 + (slice(1, -1),) * 3
    assert torch.equal(out[0], out[1]) and torch.equal(out[2][inner], ref)
    assert rel_err(f64(out[0]), conv3d.conv3d_fwd(f64(x), f64(w))) <= TOL["f32"]


@pytest.mark.parametrize("cin,cout,dtype", [(5, 7, "f32"), (48, 20, "f32"), (24, 6, "bf16"), (130, 600, "f32"), (130, 40, "bf16"),
                                              (256, 600, "bf16")])
def test_extent_one_kernels(cin, cout, dtype):
    n, dhw, grid, dt = 1, (4, 6, 37), (1, 2, 1), DT[dtype]
    g = sp3d.Geom(n, dhw, grid)
    x, dy = (synth.normal_volume((n,) + dhw + (c,), 91 + c, dtype) for c in (cin, cout))
    p = synth.weights(cin, cout, 93, dtype, taps=(1, 1, 1))
    Px, Pdy = (sp3d.alloc_padded(g, c, dt) for c in (cin, cout))
    sp3d.sp_partition(to_dev(x), Px, g, cin, dt)
    sp3d.sp_partition(to_dev(dy), Pdy, g, cout, dt)
    Py, Pdx = (sp3d.alloc_padded(g, c, dt) for c in (cout, cin))
    sp3d.sp_pointwise_fwd(Px, to_dev(p), None, Py, g, cin, cout, dt)
    sp3d.sp_pointwise_dgrad(Pdy, to_dev(p), Pdx, g, cin, cout, dt)
    dp = torch.empty((cin, cout), device="cuda")
    db = torch.empty((cout,), device="cuda")
    sp3d.sp_pointwise_wgrad(Px, Pdy, dp, db, g, cin, cout, dt,
                            sp3d.alloc_ws(sp3d.sp_workspace_bytes(sp3d.SP_OP_POINTWISE_WGRAD, g, cin, cout, dt)))
    xv, dv, pv = widen(x), widen(dy), widen(p).reshape(cin, cout)
    inner = (slice(None),) * 4 + (slice(1, -1),) * 3

    def volume(P, c):
        V = torch.empty((n,) + dhw + (c,), dtype=P.dtype, device="cuda")
        sp3d.sp_unpartition(P, V, g, c, dt)
        return f64(V)

    assert rel_err(volume(Py, cout), xv @ pv) <= TOL[dtype] and rel_err(volume(Pdx, cin), dv @ pv.T) <= TOL[dtype]
    assert rel_err(f64(dp), np.tensordot(xv, dv, axes=((0, 1, 2, 3),) * 2)) <= 1e-5
    assert rel_err(f64(db), dv.sum(axis=(0, 1, 2, 3))) <= 1e-5
    assert int(torch.count_nonzero(Py)) == int(torch.count_nonzero(Py[inner]))      # margins stay zero


@pytest.mark.parametrize("dhw, cin, cout", [((4, 9, 13), 8, 8), ((5, 7, 9), 4, 6), ((3, 5, 7), 3, 5)])
def test_infinite_voxels_stay_infinities(dhw, cin, cout):
    """Matrix-instruction slots that stand for no tap or no voxel multiply zero by zero, never zero by a voxel: with one
    infinite value in the input and finite, non-zero weights every output is an infinity or finite, none is NaN, and the
    weight gradient is not NaN where that voxel meets a non-zero gradient only or none at all."""
    g, dt = sp3d.Geom(1, dhw, (1, 1, 1)), DT["f32"]
    x = synth.normal_volume((1,) + dhw + (cin,), 4400, "f32")
    x[0, -1, -1, -1, 0] = np.inf                        # last voxel: next to slots of bricks that stick out of the tile
    dz = np.abs(synth.normal_volume((1,) + dhw + (cout,), 4401, "f32")) + np.float32(0.5)
    w = np.abs(synth.weights(cin, cout, 4402, "f32")) + np.float32(0.01)
    ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, cin, cout, dt) for op in (0, 1, 2)))
    Px, Pz, Py = (sp3d.alloc_padded(g, c, dt) for c in (cin, cout, cout))
    sp3d.sp_partition(to_dev(x), Px, g, cin, dt)
    sp3d.sp_partition(to_dev(dz), Pz, g, cout, dt)
    sp3d.conv3d_fwd(Px, to_dev(w), None, Py, g, cin, cout, dt, 0, ws)
    Y = torch.empty((1,) + dhw + (cout,), device="cuda")
    sp3d.sp_unpartition(Py, Y, g, cout, dt)
    near = torch.zeros((1,) + dhw + (1,), dtype=torch.bool, device="cuda")
    near[0, -2:, -2:, -2:] = True                       # the voxels whose kernel covers it
    assert torch.equal(torch.isinf(Y), near.expand_as(Y)) and not torch.isnan(Y).any()
    dw = torch.zeros((3, 3, 3, cin, cout), device="cuda")
    sp3d.conv3d_wgrad(Px, Pz, dw, None, g, cin, cout, dt, ws)
    hit = torch.zeros_like(dw, dtype=torch.bool)
    hit[1:, 1:, 1:, 0] = True                           # taps through which an existing voxel reads the last one
    assert torch.equal(torch.isinf(dw), hit) and not torch.isnan(dw).any()


def one_voxel(c):
    """geometry, (x, dz) in padded tiles, their values"""
    g = sp3d.Geom(1, (1, 1, 1), (1, 1, 1))
    v = [to_dev(synth.normal_volume((1, 1, 1, 1, c), 4500 + i, "f32")) for i in (0, 1)]
    P = [sp3d.alloc_padded(g, c, sp3d.SP_F32) for _ in v]
    for V, p in zip(v, P):
        sp3d.sp_partition(V, p, g, c, sp3d.SP_F32)
    return g, P, [V.view(-1) for V in v]


def test_weight_gradient_of_more_values_than_threads():
    """3600 -> 3600 channels: 350 million values, 64 to a workgroup of 1024 threads, are more threads than a launch has.  Of one
    voxel only the middle tap is not zero, and it is a product each."""
    c = 3600
    g, P, (x, dz) = one_voxel(c)
    dw, db = torch.full((27, c, c), 9.0, device="cuda"), torch.empty((c,), device="cuda")
    sp3d.conv3d_wgrad(P[0], P[1], dw, db, g, c, c, sp3d.SP_F32,
                      sp3d.alloc_ws(sp3d.sp_workspace_bytes(sp3d.SP_OP_WGRAD, g, c, c, sp3d.SP_F32)))
    assert torch.equal(dw[13], torch.outer(x, dz)) and torch.equal(db, dz)
    dw[13] = 0
    assert not dw.any()


def test_weight_gradient_of_the_widest_layers():
    """4096 -> 4096 channels: 65536 pairs of channel blocks, one more than a grid has rows."""
    c = 4096
    g, P, (x, dz) = one_voxel(c)
    dw, db = torch.empty((c, c), device="cuda"), torch.empty((c,), device="cuda")
    sp3d.sp_pointwise_wgrad(P[0], P[1], dw, db, g, c, c, sp3d.SP_F32,
                            sp3d.alloc_ws(sp3d.sp_workspace_bytes(sp3d.SP_OP_POINTWISE_WGRAD, g, c, c, sp3d.SP_F32)))
    assert torch.equal(dw, torch.outer(x, dz)) and torch.equal(db, dz)
