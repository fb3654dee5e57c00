"""The bf16 convolution kernels where a small volume makes them cut the work finer than usual: D chunks of one and two
planes with a shorter last one, with one and two input chunks per launch, with partial sums handed on between launches,
slices side by side, grown output boxes.  Bounds: one rounding of the result to bf16 (1e-2 of the value or of the rms
bounds it), fp32 sums for the weight gradient (1e-5)."""
import numpy as np
import pytest
import torch

from oracle import conv3d, flat as flat_oracle
from paper_1909_03108_amd import sp3d, synth
from gpu_util import DT, TOL, f64, rel_err, to_dev, widen

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
    (1, (9, 12, 10), (1, 2, 1), 64, 64, 1),         # 2-D: slices side by side
    (1, (7, 24, 66), (1, 1, 1), 32, 64, 1),
    (1, (5, 24, 66), (1, 2, 1), 128, 64, 1),
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
