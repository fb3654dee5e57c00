"""GPU parity of conv3d_fwd / conv3d_dgrad / conv3d_wgrad against the fp64 direct-convolution
oracle on the unpartitioned volume.  Inputs are the same stored values on both sides; the bound is
max_i |g_i - r_i| / max(|r_i|, rms(r)) <= 1e-2 for bf16 (fp32 accumulation, one bf16 rounding of the
result) and <= 1e-5 for fp32."""
import itertools

import numpy as np
import pytest
import torch

from oracle import conv3d, tiling
from paper_1909_03108_amd import sp3d, synth
from gpu_util import DT, TOL, bits, f64, rel_err, route, to_dev, widen

pytestmark = pytest.mark.gpu


class Layer:
    """Device-side plumbing for one convolution layer on a tile grid (no arithmetic here)."""

    def __init__(self, n, dhw, grid, cin, cout, dtype):
        self.g = sp3d.Geom(n, dhw, grid)
        self.cin, self.cout, self.dtype, self.dt = cin, cout, dtype, DT[dtype]
        g, dt = self.g, self.dt
        self.ws = {op: sp3d.alloc_ws(sp3d.sp_workspace_bytes(op, g, cin, cout, dt))
                   for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD, sp3d.SP_OP_WGRAD)}

    def padded(self, V, c):
        """volume (host storage array) -> halo-exchanged padded tiles on the device"""
        P = sp3d.alloc_padded(self.g, c, self.dt)
        sp3d.sp_partition(to_dev(V), P, self.g, c, self.dt)
        M = sp3d.alloc_msg(self.g, c, self.dt)
        sp3d.halo_pack(P, M, self.g, c, self.dt)
        sp3d.halo_unpack(P, M, self.g, c, self.dt)
        return P

    def volume(self, P, c):
        V = torch.empty((self.g.n, self.g.d, self.g.h, self.g.w, c), dtype=P.dtype, device="cuda")
        sp3d.sp_unpartition(P, V, self.g, c, self.dt)
        return V

    def fwd(self, x, w, bias=None, relu=False):
        Px = self.padded(x, self.cin)
        Py = sp3d.alloc_padded(self.g, self.cout, self.dt)
        b = None if bias is None else torch.from_numpy(np.asarray(bias, dtype=np.float32)).cuda()
        sp3d.conv3d_fwd(Px, to_dev(w), b, Py, self.g, self.cin, self.cout, self.dt,
                        sp3d.SP_FLAG_RELU if relu else 0, self.ws[sp3d.SP_OP_FWD])
        return self.volume(Py, self.cout)

    def dgrad(self, dz, w):
        Pz = self.padded(dz, self.cout)
        Pdx = sp3d.alloc_padded(self.g, self.cin, self.dt)
        sp3d.conv3d_dgrad(Pz, to_dev(w), Pdx, self.g, self.cin, self.cout, self.dt,
                          self.ws[sp3d.SP_OP_DGRAD])
        return self.volume(Pdx, self.cin)

    def dgrad_relu(self, dz, w, xmask):
        """data gradient with the ReLU mask of the layer input applied in the same pass"""
        Pz = self.padded(dz, self.cout)
        Pm = sp3d.alloc_padded(self.g, self.cin, self.dt)
        sp3d.sp_partition(to_dev(xmask), Pm, self.g, self.cin, self.dt)
        Pdx = sp3d.alloc_padded(self.g, self.cin, self.dt)
        sp3d.conv3d_dgrad_relu(Pz, to_dev(w), Pm, Pdx, self.g, self.cin, self.cout, self.dt,
                               self.ws[sp3d.SP_OP_DGRAD])
        return self.volume(Pdx, self.cin)

    def wgrad(self, x, dz, want_db=True):
        Px = self.padded(x, self.cin)
        Pz = sp3d.alloc_padded(self.g, self.cout, self.dt)
        sp3d.sp_partition(to_dev(dz), Pz, self.g, self.cout, self.dt)      # margins not needed
        dw = torch.full((3, 3, 3, self.cin, self.cout), 123.0, dtype=torch.float32, device="cuda")
        db = torch.full((self.cout,), 123.0, dtype=torch.float32, device="cuda") if want_db else None
        sp3d.conv3d_wgrad(Px, Pz, dw, db, self.g, self.cin, self.cout, self.dt,
                          self.ws[sp3d.SP_OP_WGRAD])
        return dw, db


def draw(dtype, shape, seed, std=1.0):
    return synth.normal_volume(shape, seed, dtype, std=std)


SMALL = [
    # n, dhw, grid, cin, cout, dtype
    (1, (8, 8, 8), (2, 2, 1), 8, 16, "f32"),
    (2, (6, 4, 10), (3, 2, 5), 3, 5, "f32"),
    (1, (3, 2, 5), (3, 2, 5), 2, 2, "bf16"),          # 1-voxel tiles
    (1, (8, 12, 16), (2, 2, 2), 1, 32, "bf16"),       # first-layer shape
    (1, (8, 16, 64), (2, 2, 1), 32, 32, "bf16"),      # the 32->32 shape, whole 8x32 patches
    (1, (12, 20, 72), (2, 2, 1), 32, 32, "bf16"),     # ragged rows and columns
    (1, (6, 10, 40), (1, 1, 2), 32, 32, "bf16"),      # split along W
    (2, (4, 8, 32), (2, 1, 1), 32, 32, "bf16"),       # batch 2
    (1, (4, 8, 16), (1, 2, 2), 64, 32, "bf16"),
    (1, (4, 8, 16), (1, 2, 2), 32, 64, "bf16"),
    (1, (5, 3, 7), (1, 1, 1), 16, 48, "bf16"),
    # input channels in multiples of 64: two chunks per launch, summed on chip (4 x 32 patches)
    (1, (16, 8, 64), (1, 2, 1), 64, 64, "bf16"),      # whole patches, 16 planes: every slot phase
    (1, (6, 8, 32), (6, 1, 1), 64, 32, "bf16"),       # one output plane per tile
    (1, (4, 12, 40), (2, 1, 1), 128, 64, "bf16"),     # two pairs (first / last), two planes, ragged
    (1, (3, 4, 32), (1, 1, 1), 192, 32, "bf16"),      # three pairs (first / middle / last), three planes
    (1, (7, 5, 33), (1, 1, 1), 64, 32, "bf16"),       # seven planes, ragged rows and columns
    # few input channels: zero-padded copies, then the matrix-core kernels
    (1, (6, 10, 40), (1, 2, 1), 3, 32, "bf16"),
    (1, (4, 8, 16), (2, 1, 1), 40, 64, "bf16"),       # 40 -> 64 channels: a pair of chunks
    # wide layers on few voxels (the bottom of a deep network): 8 and 9 launches with partial sums between them
    (1, (4, 8, 8), (1, 2, 2), 512, 128, "bf16"),      # 4 x 4 x 4 tiles
    (2, (5, 8, 6), (1, 2, 1), 576, 256, "bf16"),      # batch 2
]


@pytest.mark.parametrize("n,dhw,grid,cin,cout,dtype", SMALL)
def test_fwd_dgrad_wgrad_match_oracle(n, dhw, grid, cin, cout, dtype):
    L = Layer(n, dhw, grid, cin, cout, dtype)
    x = draw(dtype, (n,) + dhw + (cin,), 1)
    dz = draw(dtype, (n,) + dhw + (cout,), 2)
    w = synth.weights(cin, cout, 3, dtype)
    bias = np.linspace(-0.5, 0.5, cout).astype(np.float32)
    tol = TOL[dtype]

    for relu in (False, True):
        y = L.fwd(x, w, bias, relu)
        ref = conv3d.conv3d_fwd(x, widen(w), bias.astype(np.float64), relu)
        assert rel_err(f64(y), ref) <= tol, ("fwd", relu)
    dx = L.dgrad(dz, w)
    assert rel_err(f64(dx), conv3d.conv3d_dgrad(dz, widen(w))) <= tol
    dw, db = L.wgrad(x, dz)
    assert rel_err(f64(dw), conv3d.conv3d_wgrad(x, dz)) <= tol
    assert rel_err(f64(db), conv3d.bias_grad(dz)) <= tol
    # reproducible run to run (fixed-order reduction)
    dw2, db2 = L.wgrad(x, dz)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)
    dw3, none = L.wgrad(x, dz, want_db=False)
    assert none is None and torch.equal(dw, dw3)


@pytest.mark.parametrize("dtype,c", [("bf16", 32), ("f32", 4), ("bf16", 3)])
def test_identity_and_shift_kernels_are_exact_across_tile_borders(dtype, c):
    """One-hot taps copy the input shifted by tap-1 with zero fill: exact in any precision, and each
    of the 26 off-centre taps reads through a different halo region."""
    n, dhw, grid = 1, (4, 6, 64), (2, 3, 2)
    L = Layer(n, dhw, grid, c, c, dtype)
    x = draw(dtype, (n,) + dhw + (c,), 5)
    xv = widen(x)
    for tap in itertools.product(range(3), repeat=3):
        wf = np.zeros((3, 3, 3, c, c), dtype=np.float32)
        wf[tap] = np.eye(c)
        w = synth.f32_to_bf16_bits(wf) if dtype == "bf16" else wf
        y = f64(L.fwd(x, w))
        expect = np.zeros_like(xv)
        src = [slice(max(0, t - 1), e + min(0, t - 1)) for t, e in zip(tap, dhw)]
        dst = [slice(max(0, 1 - t), e + min(0, 1 - t)) for t, e in zip(tap, dhw)]
        expect[(0,) + tuple(dst)] = xv[(0,) + tuple(src)]
        assert np.array_equal(y, expect), tap
        # dgrad with the same one-hot weight shifts the other way
        dx = f64(L.dgrad(x, w))
        expect_t = np.zeros_like(xv)
        expect_t[(0,) + tuple(src)] = xv[(0,) + tuple(dst)]
        assert np.array_equal(dx, expect_t), tap


def test_outputs_touch_interiors_only():
    """conv3d_* write interior voxels; margins of the output array keep what they held."""
    n, dhw, grid, c = 1, (8, 8, 32), (2, 2, 1), 32
    L = Layer(n, dhw, grid, c, c, "bf16")
    x = draw("bf16", (n,) + dhw + (c,), 7)
    w = synth.weights(c, c, 8, "bf16")
    Px = L.padded(x, c)
    Py = torch.full(L.g.padded_shape + (c,), 3.0, dtype=torch.bfloat16, device="cuda")
    sp3d.conv3d_fwd(Px, to_dev(w), None, Py, L.g, c, c, L.dt, 0, L.ws[sp3d.SP_OP_FWD])
    got = Py.float().cpu().numpy()
    mask = np.ones(got.shape, dtype=bool)
    mask[(slice(None),) * 4 + (slice(1, -1),) * 3] = False
    assert np.all(got[mask] == 3.0)
    Pdx = torch.full(L.g.padded_shape + (c,), 3.0, dtype=torch.bfloat16, device="cuda")
    sp3d.conv3d_dgrad(Px, to_dev(w), Pdx, L.g, c, c, L.dt, L.ws[sp3d.SP_OP_DGRAD])
    assert np.all(Pdx.float().cpu().numpy()[mask] == 3.0)


def test_configuration_1_fp32_full():
    """32^3, 8 -> 16 channels, fp32, 2x2x1 grid: tiled GPU output equals the unpartitioned oracle."""
    c = synth.CONFIGS[1]
    x, ws, _ = synth.config_tensors(1)
    L = Layer(c["n"], c["dhw"], c["grid"], 8, 16, "f32")
    y = L.fwd(x, ws[0], np.zeros(16, dtype=np.float32))
    assert rel_err(f64(y), conv3d.conv3d_fwd(x, widen(ws[0]))) <= TOL["f32"]


@pytest.mark.parametrize("n,dhw,grid,cin,cout,dtype", [c for c in SMALL if c[3] > 1])
def test_dgrad_with_relu_mask_equals_dgrad_then_mask(n, dhw, grid, cin, cout, dtype):
    """conv3d_dgrad_relu = conv3d_dgrad followed by the ReLU backward on the layer input, bit for bit
    (every kernel family: one chunk, pairs, several launches, the fp32 / odd-channel direct kernel)."""
    L = Layer(n, dhw, grid, cin, cout, dtype)
    dz = draw(dtype, (n,) + dhw + (cout,), 21)
    w = synth.weights(cin, cout, 22, dtype)
    x = draw(dtype, (n,) + dhw + (cin,), 23)
    xr = np.where(widen(x) > 0, x, np.zeros_like(x))           # a ReLU output: about half zeros
    plain = L.dgrad(dz, w)
    fused = L.dgrad_relu(dz, w, xr)
    expect = torch.where(to_dev(xr).float() > 0, plain, torch.zeros_like(plain))
    assert torch.equal(fused, expect)
    assert rel_err(f64(fused), np.where(widen(xr) > 0, conv3d.conv3d_dgrad(dz, widen(w)), 0.0)) <= TOL[dtype]


SPLIT = [  # n, dhw, grid, ca, cb, cout
    (1, (8, 8, 64), (2, 1, 1), 32, 32, 32),       # one pair whose two chunks come from different tensors
    (1, (6, 12, 40), (1, 2, 1), 64, 64, 64),      # two pairs, one per tensor; ragged patches
    (1, (4, 8, 32), (1, 1, 1), 32, 64, 32),       # 96 input channels: one chunk per launch, three launches
    (2, (4, 4, 32), (2, 1, 1), 128, 128, 64),     # four pairs, batch 2
]


@pytest.mark.parametrize("n,dhw,grid,ca,cb,cout", SPLIT)
def test_two_tensor_variants_equal_concat_bit_for_bit(n, dhw, grid, ca, cb, cout):
    """conv3d_fwd2 / conv3d_dgrad2 / conv3d_wgrad2 work on concat(a, b) without materialising it: same bits as
    concatenating (or splitting) on the device and calling the single-tensor entry points."""
    g = sp3d.Geom(n, dhw, grid)
    dt, cin = sp3d.SP_BF16, ca + cb
    L = Layer(n, dhw, grid, cin, cout, "bf16")
    xa, xb = draw("bf16", (n,) + dhw + (ca,), 31), draw("bf16", (n,) + dhw + (cb,), 32)
    dz = draw("bf16", (n,) + dhw + (cout,), 33)
    w_h = synth.weights(cin, cout, 34, "bf16")
    w = to_dev(w_h)
    Pa, Pb, Pz = L.padded(xa, ca), L.padded(xb, cb), L.padded(dz, cout)
    Pc = sp3d.alloc_padded(g, cin, dt)
    sp3d.sp_concat(Pa, ca, Pb, cb, Pc, g, dt)
    ws = {op: sp3d.alloc_ws(sp3d.sp_workspace_bytes(op, g, cin, cout, dt)) for op in (0, 1, 2)}
    bias = torch.linspace(-0.5, 0.5, cout, device="cuda")
    # forward
    y1, y2 = sp3d.alloc_padded(g, cout, dt), sp3d.alloc_padded(g, cout, dt)
    sp3d.conv3d_fwd(Pc, w, bias, y1, g, cin, cout, dt, sp3d.SP_FLAG_RELU, ws[0])
    sp3d.conv3d_fwd2(Pa, ca, Pb, cb, w, bias, y2, g, cout, dt, sp3d.SP_FLAG_RELU, ws[0])
    assert torch.equal(y1, y2)
    ref = conv3d.conv3d_fwd(np.concatenate([xa, xb], axis=-1), widen(w_h), bias.double().cpu().numpy(), True)
    assert rel_err(f64(L.volume(y2, cout)), ref) <= TOL["bf16"]
    # data gradient into two tensors
    dc = sp3d.alloc_padded(g, cin, dt)
    sp3d.conv3d_dgrad(Pz, w, dc, g, cin, cout, dt, ws[1])
    da, db_ = sp3d.alloc_padded(g, ca, dt), sp3d.alloc_padded(g, cb, dt)
    sp3d.conv3d_dgrad2(Pz, w, da, ca, db_, cb, g, cout, dt, ws[1])
    ea, eb = sp3d.alloc_padded(g, ca, dt), sp3d.alloc_padded(g, cb, dt)
    sp3d.sp_split(dc, ea, ca, eb, cb, g, dt)
    assert torch.equal(L.volume(da, ca), L.volume(ea, ca)) and torch.equal(L.volume(db_, cb), L.volume(eb, cb))
    # weight gradient
    dw1 = torch.empty((3, 3, 3, cin, cout), dtype=torch.float32, device="cuda")
    dw2, b1, b2 = torch.empty_like(dw1), torch.empty(cout, device="cuda"), torch.empty(cout, device="cuda")
    sp3d.conv3d_wgrad(Pc, Pz, dw1, b1, g, cin, cout, dt, ws[2])
    sp3d.conv3d_wgrad2(Pa, ca, Pb, cb, Pz, dw2, b2, g, cout, dt, ws[2])
    assert torch.equal(dw1, dw2) and torch.equal(b1, b2)


def test_two_tensor_variants_reject_what_they_cannot_do():
    g = sp3d.Geom(1, (4, 4, 8), (1, 1, 1))
    a = sp3d.alloc_padded(g, 16, sp3d.SP_BF16)
    y = sp3d.alloc_padded(g, 32, sp3d.SP_BF16)
    w = torch.zeros((3, 3, 3, 32, 32), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(sp3d.Sp3dError) as e:
        sp3d.conv3d_fwd2(a, 16, a, 16, w, None, y, g, 32, sp3d.SP_BF16, 0, None)
    assert e.value.code == sp3d.SP_EUNSUPPORTED


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
@pytest.mark.parametrize("cin,cout,flat", [(32, 32, 0), (64, 64, 0), (32, 32, 1), (64, 64, 1), (96, 32, 0), (128, 32, 1),
                                           (32, 96, 1), (32, 128, 0), (128, 64, 0), (192, 32, 0)])
def test_every_march_length_with_mask_and_partial_sums(d, cin, cout, flat):
    """Whole patches (the marches that fetch mask values a step ahead into alternating register sets, and keep
    partial sums in fragment order) for every length of the D march modulo the slot and set periods: the masked
    data gradient equals the plain one followed by the mask, bit for bit, and the oracle within tolerance; layers
    with several launches (96, 128 and 192 kernel input channels, in the forward pass or - with the mask in the last
    launch - in the data gradient) match the oracle too.  The two-chunk kernel's march ends with two steps that
    fall on every phase of its five accumulator slots and on either register set as the length runs from 1 to 10."""
    n, dhw, grid = 1, (d, 8, 32), (1, 1, 1)
    g = sp3d.Geom(n, dhw, grid, 1, 0, flat)
    dt = DT["bf16"]
    ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, cin, cout, dt) for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD)))
    taps = (3, 3) if flat else (3, 3, 3)
    x = draw("bf16", (n,) + dhw + (cin,), 31)
    dz = draw("bf16", (n,) + dhw + (cout,), 32)
    w = synth.weights(cin, cout, 33, "bf16", taps=taps)
    xr = np.where(widen(x) > 0, x, np.zeros_like(x))

    def padded(V, c):
        P = sp3d.alloc_padded(g, c, dt)
        sp3d.sp_partition(to_dev(V), P, g, c, dt)
        sp3d.sp_halo_exchange(P, g, c, dt)
        return P

    def volume(P, c):
        V = torch.empty((n,) + dhw + (c,), dtype=P.dtype, device="cuda")
        sp3d.sp_unpartition(P, V, g, c, dt)
        return V

    if flat:
        from oracle import flat as O2
        ref_y = O2.conv_fwd(widen(x), widen(w), relu=True)
        ref_dx = O2.conv_dgrad(widen(dz), widen(w))
    else:
        ref_y = conv3d.conv3d_fwd(x, widen(w), None, True)
        ref_dx = conv3d.conv3d_dgrad(dz, widen(w))
    Px, Pz, Pm = padded(x, cin), padded(dz, cout), padded(xr, cin)
    Py = sp3d.alloc_padded(g, cout, dt)
    sp3d.conv3d_fwd(Px, to_dev(w), None, Py, g, cin, cout, dt, sp3d.SP_FLAG_RELU, ws)
    assert rel_err(f64(volume(Py, cout)), ref_y) <= TOL["bf16"]
    Pd, Pf = sp3d.alloc_padded(g, cin, dt), sp3d.alloc_padded(g, cin, dt)
    sp3d.conv3d_dgrad(Pz, to_dev(w), Pd, g, cin, cout, dt, ws)
    sp3d.conv3d_dgrad_relu(Pz, to_dev(w), Pm, Pf, g, cin, cout, dt, ws)
    plain, fused = volume(Pd, cin), volume(Pf, cin)
    assert rel_err(f64(plain), ref_dx) <= TOL["bf16"]
    assert torch.equal(fused, torch.where(to_dev(xr).float() > 0, plain, torch.zeros_like(plain)))


@pytest.mark.parametrize("grid", [(1, 8, 2), (1, 4, 6), (1, 1, 3)])     # rows of 5, 10, 40; columns of 48, 16, 32
@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 32), (96, 32), (128, 64)])
def test_patches_cut_by_the_box_give_the_bits_of_whole_ones(grid, cin, cout):
    """A march over patches that reach out of their tile's box drops the stores of the lanes outside and reads mask and partial
    sums without a condition.  Every voxel's sum is the same sum in the same order whatever the tiles, so the results of a tiling
    into such patches are, bit for bit, those of the volume as one tile, whose patches are whole: forward with bias and ReLU and
    with the mask bits written, and the data gradient masked by a tensor and by bits.  What lies outside the boxes keeps its bits."""
    n, dhw, dt = 1, (9, 40, 96), DT["bf16"]
    x, dz = draw("bf16", (n,) + dhw + (cin,), 61), draw("bf16", (n,) + dhw + (cout,), 62)
    xm = draw("bf16", (n,) + dhw + (cin,), 63)
    w, b = to_dev(synth.weights(cin, cout, 64, "bf16")), torch.linspace(-0.5, 0.5, cout, device="cuda")

    def run(gr):
        g = sp3d.Geom(n, dhw, gr)
        for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD):
            assert route(op, g, cin, cout, dt)[0] == "march"
        ws = sp3d.alloc_ws(max(sp3d.sp_workspace_bytes(op, g, cin, cout, dt) for op in (sp3d.SP_OP_FWD, sp3d.SP_OP_DGRAD)))

        def padded(V, c):
            P = sp3d.alloc_padded(g, c, dt)
            sp3d.sp_partition(to_dev(V), P, g, c, dt)
            sp3d.sp_halo_exchange(P, g, c, dt)
            return P

        def out(c):
            P = sp3d.alloc_padded(g, c, dt)
            P.fill_(7.0)
            return P

        def volume(P, c):
            keep = torch.ones(P.shape, dtype=torch.bool, device="cuda")
            keep[..., 1:-1, 1:-1, 1:-1, :] = False
            assert bool((P[keep] == 7.0).all())
            V = torch.empty((n,) + dhw + (c,), dtype=P.dtype, device="cuda")
            sp3d.sp_unpartition(P, V, g, c, dt)
            return V

        Px, Pz, Pm = padded(x, cin), padded(dz, cout), padded(xm, cin)
        words = torch.empty(sp3d.sp_relu_bits_bytes(g, cout) // 2, dtype=torch.int16, device="cuda").fill_(0x5a5a)
        want = torch.empty_like(words)
        mwords = torch.empty(sp3d.sp_relu_bits_bytes(g, cin) // 2, dtype=torch.int16, device="cuda")
        ys, ds = [out(cout), out(cout)], [out(cin), out(cin), out(cin)]
        sp3d.conv3d_fwd(Px, w, b, ys[0], g, cin, cout, dt, sp3d.SP_FLAG_RELU, ws)
        sp3d.conv3d_fwd_bits(Px, w, b, ys[1], words, g, cin, cout, dt, sp3d.SP_FLAG_RELU, ws)
        sp3d.sp_relu_bits(ys[1], want, g, cout, dt)
        words, want = (t.view(tuple(ys[0].shape[:-1]) + (cout // 32, 2)) for t in (words, want))
        inside = torch.zeros(words.shape, dtype=torch.bool, device="cuda")
        inside[..., 1:-1, 1:-1, 1:-1, :, :] = True
        assert torch.equal(words, torch.where(inside, want, torch.full_like(want, 0x5a5a)))
        sp3d.sp_relu_bits(Pm, mwords, g, cin, dt)
        sp3d.conv3d_dgrad(Pz, w, ds[0], g, cin, cout, dt, ws)
        sp3d.conv3d_dgrad_relu(Pz, w, Pm, ds[1], g, cin, cout, dt, ws)
        sp3d.conv3d_dgrad_bits(Pz, w, mwords, ds[2], g, cin, cout, dt, ws)
        return [volume(P, cout) for P in ys] + [volume(P, cin) for P in ds]

    whole, cut = run((1, 1, 1)), run(grid)
    for a, c in zip(whole, cut):
        assert torch.equal(a, c)
    assert torch.equal(whole[3], whole[4])
