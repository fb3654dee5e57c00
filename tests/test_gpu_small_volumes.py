"""The bf16 convolution kernels where a small volume makes them cut the work finer than usual: D chunks of one and two
planes with a shorter last one, with one and two input chunks per launch, with partial sums handed on between launches,
slices side by side, grown output boxes.  Bounds: one rounding of the result to bf16 (1e-2 of the value or of the rms
bounds it), fp32 sums for the weight gradient (1e-5)."""
import numpy as np
import pytest
import torch

from oracle import conv3d, flat as flat_oracle
from paper_1909_03108_amd import sp3d, synth
from gpu_util import DT, TOL, f64, rel_err, route, to_dev, widen
from test_gpu_gather import test_gathered_halos_equal_exchange_then_convolve as check_gathered_halos
from test_gpu_relu_bits import test_convolutions_write_and_read_the_bits as check_bits

pytestmark = pytest.mark.gpu


def three_passes(n, dhw, grid, cin, cout, flat, seed):
    """forward with bias and ReLU, masked and plain data gradient, weight gradient against the oracle"""
    dt, tol = DT["bf16"], TOL["bf16"]
    g = sp3d.Geom(n, dhw, grid, 1, 0, flat)
    x = synth.normal_volume((n,) + dhw + (cin,), seed, "bf16")
    dz = synth.normal_volume((n,) + dhw + (cout,), seed + 1, "bf16")
    w = synth.weights(cin, cout, seed + 2, "bf16", taps=(3, 3) if flat else (3, 3, 3))
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
    assert torch.equal(dw, again)
    xv, zv, wv, bv = widen(x), widen(dz), widen(w), bias.astype(np.float64)
    O = flat_oracle if flat else conv3d
    y, dx, rw, rb = ((O.conv_fwd(xv, wv, bv, True), O.conv_dgrad(zv, wv), O.conv_wgrad(xv, zv), O.bias_grad(zv)) if flat else
                     (O.conv3d_fwd(x, wv, bv, True), O.conv3d_dgrad(dz, wv), O.conv3d_wgrad(x, dz), O.bias_grad(dz)))
    assert rel_err(volume(Py, cout), y) <= tol
    assert rel_err(volume(Pdx, cin), dx) <= tol
    assert np.array_equal(volume(Pdm, cin), np.where(xv > 0, volume(Pdx, cin), 0.0))
    assert rel_err(f64(dw), rw) <= 1e-5 and rel_err(f64(db), rb) <= 1e-5


CHUNKS = [  # n, dhw, grid, cin, cout, flat
    (1, (5, 8, 32), (1, 1, 1), 32, 32, 0),          # chunks of one plane
    (1, (14, 9, 34), (2, 1, 1), 32, 64, 0),         # ... ragged patches, several output blocks
    (1, (7, 6, 20), (1, 1, 1), 64, 32, 0),          # two input chunks per launch
    (1, (22, 16, 32), (1, 2, 1), 128, 32, 0),       # ... and partial sums (first and last launch)
    (1, (33, 40, 70), (1, 1, 1), 192, 96, 0),       # ... a middle launch; chunks of several planes, a shorter last one
    (1, (9, 12, 10), (1, 2, 1), 64, 64, 1),
    (1, (7, 24, 66), (1, 1, 1), 32, 64, 1),
    (1, (5, 24, 66), (1, 2, 1), 128, 64, 1),
    (1, (8, 12, 10), (1, 2, 1), 32, 64, 1),         # 2-D: two and three slices side by side
    (2, (6, 9, 9), (1, 1, 1), 64, 32, 1),
]


@pytest.mark.parametrize("case", CHUNKS, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_short_marches(case):
    three_passes(*case, seed=5100 + 10 * CHUNKS.index(case))


GEMM = [  # wide layers: the implicit GEMM (conv_gemm.hip); dhw and grid set the row length its record loads are sized for
    (1, (1, 1, 1), (1, 1, 1), 512, 512, 0),
    (2, (3, 5, 1), (1, 1, 1), 512, 512, 0),         # rows of 1 voxel: 3 records per voxel
    (1, (4, 6, 4), (2, 2, 2), 512, 512, 0),         # 2
    (1, (3, 7, 3), (1, 1, 1), 576, 512, 0),         # 3; 18 input chunks
    (1, (5, 6, 13), (1, 3, 1), 512, 512, 0),
    (1, (2, 3, 70), (1, 1, 1), 512, 512, 0),
    (3, (2, 10, 140), (1, 1, 1), 512, 512, 1),      # 2-D; rows longer than a tile of 128 voxels
    (1, (16, 28, 28), (1, 4, 4), 512, 512, 1),      # 256 voxels per workgroup, rows of 7
]


@pytest.mark.parametrize("case", GEMM, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_wide_layers_on_few_voxels(case):
    three_passes(*case, seed=5300 + 10 * GEMM.index(case))


NARROW_GEMM = [  # layers the implicit GEMM takes over from the marching kernels: one and two output blocks per wave,
                 # input chunks odd in number, both voxel tiles, every count of record loads, one and several splits
    (1, (4, 6, 1), (2, 2, 1), 128, 64, 0),
    (1, (5, 6, 9), (1, 2, 3), 96, 192, 0),
    (2, (8, 12, 14), (2, 2, 2), 160, 64, 0),
    (1, (17, 24, 33), (1, 1, 1), 128, 64, 0),
    (1, (3, 130, 70), (1, 1, 2), 192, 64, 1),
    (1, (1, 96, 200), (1, 2, 1), 64, 128, 1),
    (1, (2, 256, 182), (1, 2, 26), 128, 64, 1),     # rows of 7 voxels in tiles of 256
    (1, (2, 256, 256), (1, 2, 2), 128, 128, 1),     # several workgroups per compute unit, no split
]


@pytest.mark.parametrize("case", NARROW_GEMM, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_layers_taken_over_by_the_implicit_gemm(case):
    three_passes(*case, seed=5500 + 10 * NARROW_GEMM.index(case))


SEVERAL_ITEMS = [  # more tiles than workgroups that fit on the chip, not a multiple of them: a workgroup goes from one to the next
    (1, (5, 120, 126), (1, 2, 2), 128, 128, 1),     # 591 tiles, 512 workgroups
    (1, (11, 190, 70), (1, 1, 2), 96, 64, 1),       # 572, three chunks
    (1, (27, 60, 70), (1, 1, 2), 96, 128, 0),       # 443, 256 workgroups
    (1, (1, 300, 260), (1, 1, 2), 32, 128, 1),      # 610 of three steps: the loads run ahead by most of an item
]


@pytest.mark.parametrize("case", SEVERAL_ITEMS, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_several_tiles_per_workgroup(case):
    n, dhw, grid, cin, cout, flat = case
    family, (cbw, vb, _, splits) = route(sp3d.SP_OP_FWD, sp3d.Geom(n, dhw, grid, 1, 0, flat), cin, cout, sp3d.SP_BF16)
    items = -(-dhw[0] * dhw[1] * dhw[2] // (128 * vb)) * (cout // (64 * cbw))
    assert family == "gemm" and splits == 1 and items % 256 and items > (256 if (cbw, vb) == (2, 2) else 512)
    three_passes(*case, seed=7100 + 10 * SEVERAL_ITEMS.index(case))


ROWS = [  # 2-D, 32 and 64 input channels (conv_rows2d.hip): one row, strips of 1 ... 32 columns, fewer rows than the ring holds and one
         # more, chunks with a shorter last one, several blocks of output channels
    (1, (1, 1, 16), (1, 1, 1), 32, 32, 1),
    (2, (3, 2, 33), (1, 1, 1), 32, 64, 1),
    (1, (2, 7, 64), (1, 1, 2), 32, 32, 1),
    (1, (3, 27, 40), (1, 3, 2), 32, 96, 1),
    (1, (1, 301, 97), (1, 1, 1), 32, 32, 1),
    (1, (16, 86, 65), (1, 2, 1), 32, 64, 1),
    (1, (1, 1, 16), (1, 1, 1), 64, 32, 1),
    (1, (3, 27, 40), (1, 3, 2), 64, 96, 1),
    (1, (16, 100, 66), (1, 2, 1), 64, 64, 1),
]


@pytest.mark.parametrize("case", ROWS, ids=lambda c: "%dx%dx%d-%dto%d" % (c[1] + c[3:5]))
def test_row_marches(case):
    three_passes(*case, seed=7300 + 10 * ROWS.index(case))


@pytest.mark.parametrize("c", [32, 64])
def test_row_and_patch_marches_give_the_same_bits(c):
    """Tiles of 15 columns lie side by side in a patch (conv_mfma.hip, conv_mfma_pair_kernel.h), one of 30 is a strip of rows."""
    dhw, dt = (4, 21, 30), DT["bf16"]
    x, z = (to_dev(synth.normal_volume((1,) + dhw + (c,), 7400 + i, "bf16")) for i in (0, 1))
    w = to_dev(synth.weights(c, c, 7402, "bf16", taps=(3, 3)))
    res = []
    for grid in ((1, 1, 2), (1, 1, 1)):
        g = sp3d.Geom(1, dhw, grid, 1, 0, 1)
        assert {route(op, g, c, c, dt)[0] for op in (0, 1)} == {"march"}
        ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, c, c, dt) for op in (0, 1)))
        P, Z, Y, D = (sp3d.alloc_padded(g, c, dt) for _ in range(4))
        for V, T in ((x, P), (z, Z)):
            sp3d.sp_partition(V, T, g, c, dt)
            sp3d.sp_halo_exchange(T, g, c, dt)
        sp3d.conv3d_fwd(P, w, None, Y, g, c, c, dt, sp3d.SP_FLAG_RELU, ws)
        sp3d.conv3d_dgrad_relu(Z, w, P, D, g, c, c, dt, ws)
        out = [torch.empty_like(x) for _ in range(2)]
        sp3d.sp_unpartition(Y, out[0], g, c, dt)
        sp3d.sp_unpartition(D, out[1], g, c, dt)
        res.append(out)
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


SPLIT_TILES = [  # tiles of 256 voxels and several splits: both numbers of output blocks per wave, whole and ragged last tiles
    (1, (5, 32, 32), (1, 2, 2), 512, 512, 1),
    (1, (5, 33, 31), (1, 1, 1), 512, 512, 1),
    (1, (2, 96, 96), (1, 2, 2), 256, 64, 0),
    (1, (2, 94, 98), (1, 2, 2), 256, 64, 0),
]


@pytest.mark.parametrize("case", SPLIT_TILES, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_split_sums_of_the_larger_tiles(case):
    three_passes(*case, seed=6700 + 10 * SPLIT_TILES.index(case))


@pytest.mark.parametrize("n, dhw, grid, cin, cout", [(1, (4, 4, 4), (4, 2, 2), 128, 128), (2, (6, 5, 9), (2, 1, 3), 192, 64),
                                                     (1, (12, 18, 10), (3, 3, 2), 128, 256)])
def test_implicit_gemm_gathers_halos_and_keeps_bits(n, dhw, grid, cin, cout):
    check_gathered_halos(n, dhw, grid, cin, cout)
    check_bits(n, dhw, grid, cin, cout)


GROWN = [  # dhw, grid, ca, cb, cout: input in two tensors; output as well; tiles of 256 voxels with several splits
    ((8, 10, 14), (2, 2, 2), 96, 64, 192),
    ((8, 10, 14), (2, 2, 2), 96, 96, 192),
    ((2, 96, 96), (1, 2, 2), 160, 96, 64),
]


@pytest.mark.parametrize("dhw, grid, ca, cb, co", GROWN)
def test_implicit_gemm_grown_boxes_and_two_tensors(dhw, grid, ca, cb, co):
    """A grown output box on margins two voxels wide, input and output in two tensors, at odd chunk counts: bit for bit
    what the one-voxel margins, the concatenation and the single tensor give."""
    n, dt = 1, DT["bf16"]
    g1, g2 = sp3d.Geom(n, dhw, grid), sp3d.Geom(n, dhw, grid, 2, 1)
    x = synth.normal_volume((n,) + dhw + (ca + cb,), 5700, "bf16")
    dz = synth.normal_volume((n,) + dhw + (co,), 5701, "bf16")
    w = to_dev(synth.weights(ca + cb, co, 5702, "bf16"))

    def padded(g, v, c):
        P = sp3d.alloc_padded(g, c, dt)
        sp3d.sp_partition(to_dev(np.ascontiguousarray(v)), P, g, c, dt)
        sp3d.sp_halo_exchange(P, g, c, dt)
        return P

    def volume(g, P, c):
        V = torch.empty((n,) + dhw + (c,), dtype=torch.bfloat16, device="cuda")
        sp3d.sp_unpartition(P, V, g, c, dt)
        return V

    res = []
    for g in (g1, g2):
        ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, ca + cb, co, dt) for op in (0, 1)))
        P, Pa, Pb, Z = padded(g, x, ca + cb), padded(g, x[..., :ca], ca), padded(g, x[..., ca:], cb), padded(g, dz, co)
        Y, Y2, D = (sp3d.alloc_padded(g, c, dt) for c in (co, co, ca + cb))
        Da, Db = sp3d.alloc_padded(g, ca, dt), sp3d.alloc_padded(g, cb, dt)
        sp3d.conv3d_fwd(P, w, None, Y, g, ca + cb, co, dt, sp3d.SP_FLAG_RELU, ws)
        sp3d.conv3d_fwd2(Pa, ca, Pb, cb, w, None, Y2, g, co, dt, sp3d.SP_FLAG_RELU, ws)
        sp3d.conv3d_dgrad(Z, w, D, g, ca + cb, co, dt, ws)
        sp3d.conv3d_dgrad2(Z, w, Da, ca, Db, cb, g, co, dt, ws)
        assert torch.equal(Y, Y2)
        assert torch.equal(D[..., :ca], Da) and torch.equal(D[..., ca:], Db)
        if g is g2:                                     # the surround holds what the neighbour computed for itself
            E = Y.clone()
            sp3d.sp_halo_exchange(E, g, co, dt)
            inner = (slice(None),) * 4 + (slice(1, -1),) * 3
            assert torch.equal(E[inner], Y[inner]) and bool((Y[inner] != 0).any())
        res.append((volume(g, Y, co), volume(g, D, ca + cb)))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    ref = conv3d.conv3d_fwd(x, widen(synth.weights(ca + cb, co, 5702, "bf16")), None, relu=True)
    assert rel_err(f64(res[0][0]), ref) <= TOL["bf16"]


WGRAD_GEMM = [  # weight gradients as a GEMM over voxels: both channel tiles, every count of record loads, one and several
                # splits, stages that end inside a row, a slice and a tile, a last stage of 1 ... 63 voxels
    (1, (3, 4, 2), (1, 2, 1), 64, 64, 0),           # rows of 2 voxels: 128 records a stage
    (1, (2, 2, 3), (1, 1, 1), 128, 256, 0),         # fewer voxels than a stage
    (2, (5, 6, 7), (1, 2, 1), 192, 64, 0),
    (1, (8, 8, 8), (2, 2, 2), 128, 128, 0),         # rows of 4
    (1, (9, 10, 33), (1, 1, 1), 64, 128, 0),
    (1, (3, 20, 65), (1, 1, 1), 256, 128, 1),       # a last stage of 60 voxels
    (1, (1, 9, 129), (1, 1, 1), 128, 128, 1),
    (1, (5, 40, 24), (1, 4, 4), 320, 64, 1),
]


@pytest.mark.parametrize("case", WGRAD_GEMM, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_weight_gradient_as_a_gemm(case):
    three_passes(*case, seed=5900 + 10 * WGRAD_GEMM.index(case))


WGRAD_GATHER = [  # gathered halos: both channel tiles, one running sum and a sum per stage
    ((4, 16, 64), (2, 2, 2), 64, 128), ((1, 16, 32), (1, 2, 1), 64, 64), ((1, 32, 128), (1, 2, 2), 128, 128),
    ((1, 16, 64), (1, 2, 1), 384, 384)]


def test_weight_gradient_gemm_gathers_and_takes_two_tensors():
    for dhw, grid, cin, cout in WGRAD_GATHER:
        check_gathered_halos(1, dhw, grid, cin, cout)
    n, dhw, grid, ca, cb, co, dt = 1, (4, 6, 10), (2, 2, 1), 32, 96, 64, DT["bf16"]
    g = sp3d.Geom(n, dhw, grid)
    x = synth.normal_volume((n,) + dhw + (ca + cb,), 6001, "bf16")
    dz = synth.normal_volume((n,) + dhw + (co,), 6002, "bf16")
    P = []
    for v in (x, x[..., :ca], x[..., ca:], dz):
        P.append(sp3d.alloc_padded(g, v.shape[-1], dt))
        sp3d.sp_partition(to_dev(np.ascontiguousarray(v)), P[-1], g, v.shape[-1], dt)
        sp3d.sp_halo_exchange(P[-1], g, v.shape[-1], dt)
    ws = sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, ca + cb, co, dt))
    store = torch.zeros(2 * co + 1, device="cuda")
    dw, dw2, db, db2 = torch.empty((3, 3, 3, ca + cb, co), device="cuda"), torch.empty((3, 3, 3, ca + cb, co), device="cuda"), \
        store[1:co + 1], store[co + 1:]                 # (a bias gradient may lie at any multiple of four bytes)
    sp3d.conv3d_wgrad(P[0], P[3], dw, db, g, ca + cb, co, dt, ws)
    sp3d.conv3d_wgrad2(P[1], ca, P[2], cb, P[3], dw2, db2, g, co, dt, ws)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)
    assert rel_err(f64(dw), conv3d.conv3d_wgrad(x, dz)) <= 1e-5 and rel_err(f64(db), conv3d.bias_grad(dz)) <= 1e-5


def test_weight_gradient_of_an_infinite_voxel():
    """The last stage's clamped voxels are masked in both operands: an infinity in the last voxel reaches only the taps
    and channels that read it."""
    g, dt = sp3d.Geom(1, (3, 5, 7), (1, 1, 1)), DT["bf16"]
    x = synth.normal_volume((1, 3, 5, 7, 64), 6101, "bf16")
    x[0, -1, -1, -1, 5] = 0x7f80                        # + infinity
    dz = synth.normal_volume((1, 3, 5, 7, 64), 6102, "bf16")
    Px, Pz = sp3d.alloc_padded(g, 64, dt), sp3d.alloc_padded(g, 64, dt)
    sp3d.sp_partition(to_dev(x), Px, g, 64, dt)
    sp3d.sp_partition(to_dev(dz), Pz, g, 64, dt)
    dw = torch.zeros((3, 3, 3, 64, 64), device="cuda")
    sp3d.conv3d_wgrad(Px, Pz, dw, None, g, 64, 64, dt, sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, 64, 64, dt)))
    hit = torch.zeros_like(dw, dtype=torch.bool)
    hit[1:, 1:, 1:, 5] = True
    assert torch.equal(torch.isinf(dw), hit) and not torch.isnan(dw).any()


FINE_WGRAD = [  # D chunks of the marching weight gradient: one and two planes, a shorter last one, whole and ragged patches,
                # and behind zero-padded input channels (of up to eight channels there are no copies: FEW)
    (1, (7, 8, 32), (1, 1, 1), 32, 32, 0),
    (1, (22, 16, 64), (2, 1, 2), 32, 96, 0),
    (1, (13, 9, 34), (1, 1, 1), 96, 32, 0),
    (1, (11, 6, 40), (1, 2, 1), 12, 32, 0),
    (1, (9, 12, 10), (1, 2, 1), 32, 32, 1),
    (1, (6, 16, 96), (1, 2, 1), 20, 64, 1),
    (1, (8, 12, 10), (1, 2, 1), 32, 32, 1),         # 2-D: slices side by side
    (2, (6, 9, 9), (1, 1, 1), 64, 32, 1),
]


@pytest.mark.parametrize("case", FINE_WGRAD, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_short_weight_gradient_marches(case):
    three_passes(*case, seed=6200 + 10 * FINE_WGRAD.index(case))


STATIC = [(edge, cin) for edge in (20, 40, 64) for cin in (12, 3)]      # 12: padded copies; 3: none (FEW)


@pytest.mark.parametrize("edge, cin", STATIC)
def test_static_scratch_takes_padded_layers(edge, cin):
    """Zero-padded layers share the library's own buffer between the copies and the partial results: the same bits as with
    a workspace, whichever cutting the sizes allow."""
    g, dt = sp3d.Geom(1, (edge,) * 3, (1, 1, 1)), DT["bf16"]
    x, dz = (synth.normal_volume((1,) + (edge,) * 3 + (c,), 6300 + c, "bf16") for c in (cin, 32))
    Px, Pz = sp3d.alloc_padded(g, cin, dt), sp3d.alloc_padded(g, 32, dt)
    sp3d.sp_partition(to_dev(x), Px, g, cin, dt)
    sp3d.sp_partition(to_dev(dz), Pz, g, 32, dt)
    need = sp3d.sp_workspace_bytes(2, g, cin, 32, dt)
    assert need <= sp3d.SP_STATIC_SCRATCH_BYTES
    a, b = torch.empty((3, 3, 3, cin, 32), device="cuda"), torch.empty((3, 3, 3, cin, 32), device="cuda")
    sp3d.conv3d_wgrad(Px, Pz, a, None, g, cin, 32, dt, sp3d.alloc_ws(need))
    sp3d.conv3d_wgrad_static(Px, Pz, b, None, g, cin, 32, dt)
    assert torch.equal(a, b)
    assert rel_err(f64(a), conv3d.conv3d_wgrad(x, dz)) <= 1e-5


FEW = [  # first layers of 2 ... 8 channels: both record sizes, odd channel counts, bricks that stick out, several output blocks
    (1, (1, 1, 1), (1, 1, 1), 2, 32, 0),
    (2, (5, 6, 34), (1, 2, 1), 3, 64, 0),
    (1, (9, 10, 66), (1, 2, 2), 4, 32, 0),
    (1, (4, 9, 31), (2, 1, 1), 5, 96, 0),
    (1, (10, 13, 40), (1, 1, 1), 8, 32, 0),
    (1, (3, 8, 50), (1, 2, 1), 3, 32, 1),
    (1, (7, 10, 36), (1, 2, 2), 7, 64, 1),
    (1, (1, 200, 210), (1, 1, 1), 5, 32, 1),        # several bricks per workgroup
    (1, (5, 7, 35), (1, 1, 1), 6, 32, 0),
    (1, (11, 6, 40), (1, 2, 1), 3, 32, 0),
    (1, (6, 16, 96), (1, 2, 1), 5, 64, 1),
]


@pytest.mark.parametrize("case", FEW, ids=lambda c: "%dx%dx%d-%dto%d%s" % (c[1] + c[3:5] + ("-2d" if c[5] else "",)))
def test_first_layers_of_few_channels(case):
    three_passes(*case, seed=6400 + 10 * FEW.index(case))


def test_few_channels_grown_box_and_infinities():
    """A grown output box gives what the neighbour computes for itself; an infinite voxel reaches only the outputs that
    read it (unused K slots are zero in both operands)."""
    n, dhw, grid, ci, co, dt = 1, (8, 10, 70), (2, 2, 2), 3, 32, DT["bf16"]
    x = synth.normal_volume((n,) + dhw + (ci,), 6501, "bf16")
    w = to_dev(synth.weights(ci, co, 6502, "bf16"))
    out = []
    for g in (sp3d.Geom(n, dhw, grid), sp3d.Geom(n, dhw, grid, 2, 1)):
        P, Y = sp3d.alloc_padded(g, ci, dt), sp3d.alloc_padded(g, co, dt)
        sp3d.sp_partition(to_dev(x), P, g, ci, dt)
        sp3d.sp_halo_exchange(P, g, ci, dt)
        sp3d.conv3d_fwd(P, w, None, Y, g, ci, co, dt, 0, sp3d.alloc_ws(sp3d.sp_workspace_bytes(0, g, ci, co, dt)))
        V = torch.empty((n,) + dhw + (co,), dtype=torch.bfloat16, device="cuda")
        sp3d.sp_unpartition(Y, V, g, co, dt)
        out.append(V)
    E = Y.clone()
    sp3d.sp_halo_exchange(E, g, co, dt)
    inner = (slice(None),) * 4 + (slice(1, -1),) * 3
    assert torch.equal(E[inner], Y[inner]) and torch.equal(out[0], out[1])
    g = sp3d.Geom(1, (5, 6, 33), (1, 1, 1))
    x = synth.normal_volume((1, 5, 6, 33, ci), 6503, "bf16")
    x[0, -1, -1, -1, 0] = 0x7f80                        # + infinity
    w = to_dev(np.where(widen(synth.weights(ci, co, 6504, "bf16")) == 0, np.uint16(0x3f80), synth.weights(ci, co, 6504, "bf16")))
    P, Y = sp3d.alloc_padded(g, ci, dt), sp3d.alloc_padded(g, co, dt)
    sp3d.sp_partition(to_dev(x), P, g, ci, dt)
    sp3d.conv3d_fwd(P, w, None, Y, g, ci, co, dt, 0, sp3d.alloc_ws(sp3d.sp_workspace_bytes(0, g, ci, co, dt)))
    V = torch.empty((1, 5, 6, 33, co), dtype=torch.bfloat16, device="cuda")
    sp3d.sp_unpartition(Y, V, g, co, dt)
    near = torch.zeros((1, 5, 6, 33, 1), dtype=torch.bool, device="cuda")
    near[0, -2:, -2:, -2:] = True
    assert torch.equal(torch.isinf(V), near.expand_as(V)) and not torch.isnan(V).any()


FLAT_PATCHES = [(1, (4, 16, 64), (1, 2, 1), 32, 64, 32), (2, (1, 8, 96), (1, 1, 1), 64, 32, 64), (1, (5, 104, 96), (1, 1, 1), 160, 96, 32),
                (1, (9, 120, 96), (1, 5, 1), 32, 64, 64)]


@pytest.mark.parametrize("n, dhw, grid, ca, cb, co", FLAT_PATCHES)
def test_flat_whole_patches_take_two_tensors(n, dhw, grid, ca, cb, co):
    """The weight gradient of whole patches in 2-D with its input channels in two tensors: the bits of one tensor."""
    g, dt = sp3d.Geom(n, dhw, grid, 1, 0, 1), DT["bf16"]
    x = synth.normal_volume((n,) + dhw + (ca + cb,), 6701, "bf16")
    dz = synth.normal_volume((n,) + dhw + (co,), 6702, "bf16")
    P = []
    for v in (x, x[..., :ca], x[..., ca:], dz):
        P.append(sp3d.alloc_padded(g, v.shape[-1], dt))
        sp3d.sp_partition(to_dev(np.ascontiguousarray(v)), P[-1], g, v.shape[-1], dt)
        sp3d.sp_halo_exchange(P[-1], g, v.shape[-1], dt)
    ws = sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, ca + cb, co, dt))
    dw, dw2 = torch.empty((3, 3, ca + cb, co), device="cuda"), torch.empty((3, 3, ca + cb, co), device="cuda")
    db, db2 = torch.empty(co, device="cuda"), torch.empty(co, device="cuda")
    sp3d.conv3d_wgrad(P[0], P[3], dw, db, g, ca + cb, co, dt, ws)
    sp3d.conv3d_wgrad2(P[1], ca, P[2], cb, P[3], dw2, db2, g, co, dt, ws)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)
    assert rel_err(f64(dw), flat_oracle.conv_wgrad(widen(x), widen(dz))) <= 1e-5
    assert rel_err(f64(db), flat_oracle.bias_grad(widen(dz))) <= 1e-5


# 64 x 64 channels to a workgroup: blocks whose two halves lie in different tensors, an odd number of input blocks, several tiles and
# entries, workgroups with a unit less than others, in one pass and in two (units, workgroups per block: 768, 112; 144, 37; 256, 18;
# 357, 37)
FLAT_BLOCKS = [(2, (6, 128, 128), (1, 2, 2), 32, 96, 64), (1, (4, 96, 96), (1, 1, 1), 96, 96, 128),
               (1, (16, 64, 64), (1, 2, 1), 224, 32, 192), (1, (7, 136, 96), (1, 1, 1), 96, 96, 128)]


@pytest.mark.parametrize("n, dhw, grid, ca, cb, co", FLAT_BLOCKS)
def test_flat_blocks_of_four_pairs(n, dhw, grid, ca, cb, co):
    """Four channel pairs per workgroup: the oracle's sums, the same bits from two tensors and without the bias gradient, and with
    NaN in whatever lies outside (margins along D, workspace)."""
    g, dt = sp3d.Geom(n, dhw, grid, 1, 0, 1), DT["bf16"]
    family, detail = route(2, g, ca + cb, co, dt)
    assert family == "march" and detail[0] == 2 and detail[3] * (ca + cb) * co > 256 * 32 * 32
    x = synth.normal_volume((n,) + dhw + (ca + cb,), 6711, "bf16")
    dz = synth.normal_volume((n,) + dhw + (co,), 6712, "bf16")
    P = []
    for v in (x, x[..., :ca], x[..., ca:], dz):
        P.append(sp3d.alloc_padded(g, v.shape[-1], dt))
        P[-1][..., 0, :, :, :] = P[-1][..., -1, :, :, :] = float("nan")
        sp3d.sp_partition(to_dev(np.ascontiguousarray(v)), P[-1], g, v.shape[-1], dt)
        sp3d.sp_halo_exchange(P[-1], g, v.shape[-1], dt)
    ws = sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, ca + cb, co, dt))
    ws.fill_(255)
    dw, dw2, dw3 = (torch.empty((3, 3, ca + cb, co), device="cuda") for _ in range(3))
    db, db2 = torch.empty(co, device="cuda"), torch.empty(co, device="cuda")
    sp3d.conv3d_wgrad(P[0], P[3], dw, db, g, ca + cb, co, dt, ws)
    sp3d.conv3d_wgrad2(P[1], ca, P[2], cb, P[3], dw2, db2, g, co, dt, ws)
    sp3d.conv3d_wgrad(P[0], P[3], dw3, None, g, ca + cb, co, dt, ws)
    assert torch.equal(dw, dw2) and torch.equal(db, db2) and torch.equal(dw, dw3)
    assert rel_err(f64(dw), flat_oracle.conv_wgrad(widen(x), widen(dz))) <= 1e-5
    assert rel_err(f64(db), flat_oracle.bias_grad(widen(dz))) <= 1e-5


@pytest.mark.parametrize("cin", [3, 6])                 # records of 4 and of 8 channels
@pytest.mark.parametrize("flat", [0, 1])
@pytest.mark.parametrize("tiles", [1, 2])
def test_few_channel_weight_gradient_of_an_infinite_voxel(cin, flat, tiles):
    """Rows of 33 voxels end one voxel into their second brick; what lies behind is masked in both operands (dz alone would turn
    the infinity into NaN), and the rows past the last channel of a kernel row are dropped: an infinity in the last voxel, or in
    the first of the next tile, reaches only the taps and the channel that read it."""
    g, dt, co = sp3d.Geom(1, (5, 6, 33 * tiles), (1, 1, tiles), 1, 0, flat), DT["bf16"], 32
    x, dz = (synth.normal_volume((1, 5, 6, 33 * tiles, c), 6600 + c, "bf16") for c in (cin, co))
    for a in (x, dz):
        a[widen(a) == 0] = 0x3f80
    x[0, -1, -1, 32 if tiles == 1 else 33, cin - 1] = 0x7f80          # + infinity
    Px, Pz = sp3d.alloc_padded(g, cin, dt), sp3d.alloc_padded(g, co, dt)
    sp3d.sp_partition(to_dev(x), Px, g, cin, dt)
    sp3d.sp_halo_exchange(Px, g, cin, dt)
    sp3d.sp_partition(to_dev(dz), Pz, g, co, dt)
    dw, db = torch.empty((1 if flat else 3, 3, 3, cin, co), device="cuda"), torch.empty((co,), device="cuda")
    sp3d.conv3d_wgrad(Px, Pz, dw, db, g, cin, co, dt, sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, cin, co, dt)))
    hit = torch.zeros_like(dw, dtype=torch.bool)
    hit[0 if flat else 1:, 1:, 1 if tiles == 1 else 0:, cin - 1] = True
    assert torch.equal(torch.isinf(dw), hit) and not torch.isnan(dw).any()
    assert rel_err(f64(db), widen(dz).reshape(-1, co).sum(0)) <= 1e-5
