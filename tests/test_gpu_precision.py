"""Weight gradients against 64 bits: the error of the fp32 sums, in the 2-norm over the 2-norm of the result.

Bounds.  A rounding of a running sum s is off by at most 2^-24 |s|, by 2^-24 |s| / sqrt(3) in the root mean square; where
products of random sign are added, s grows like the square root of their number, so that a chain of n roundings ends
sqrt(n / 2) 2^-24 / sqrt(3) off the result.  The reference is the
same sum tap by tap in torch's float64."""
import math

import pytest
import torch

from paper_1909_03108_amd import sp3d, synth
from gpu_util import DT, route, to_dev

pytestmark = pytest.mark.gpu


def chain(n):
    return math.sqrt(n / 6) * 2.0 ** -24


def off(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


def weight_gradient(n, dhw, grid, cin, cout, dtype, flat, seed=7100):
    """errors of dw and db"""
    g, dt = sp3d.Geom(n, dhw, grid, 1, 0, flat), DT[dtype]
    x, dz = (to_dev(synth.normal_volume((n,) + dhw + (c,), seed + i, dtype)) for i, c in enumerate((cin, cout)))
    P = []
    for v, c in ((x, cin), (dz, cout)):
        P.append(sp3d.alloc_padded(g, c, dt))
        sp3d.sp_partition(v, P[-1], g, c, dt)
        sp3d.sp_halo_exchange(P[-1], g, c, dt)
    dw = torch.empty((9 if flat else 27, cin, cout), device="cuda")
    db = torch.empty((cout,), device="cuda")
    sp3d.conv3d_wgrad(P[0], P[1], dw, db, g, cin, cout, dt, sp3d.alloc_ws(sp3d.sp_workspace_bytes(2, g, cin, cout, dt)))
    D, H, W = dhw
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1) + ((0, 0) if flat else (1, 1)))
    z = dz.double().reshape(-1, cout)
    ref = torch.stack([xp[:, a:a + D, b:b + H, c:c + W].reshape(-1, cin).t() @ z
                       for a in range(1 if flat else 3) for b in range(3) for c in range(3)])
    return off(dw, ref), off(db, z.sum(0))


# As a GEMM over voxels, summed by stage: each split adds its stages of 64 voxels to a running sum, 36 of them at most in these
# layers; inside a stage the sums of up to 64 voxels are rounded at most 16 times: chain(36 + 16 / 2).  (With running sums
# that every product was added to: 2.2e-7, 2.8e-7, 2.0e-7; bias gradient of the third 7.4e-8.)
@pytest.mark.parametrize("n, dhw, grid, cin, cout, flat", [
    (1, (18, 16, 16), (1, 1, 4), 512, 64, 0), (1, (17, 24, 22), (1, 2, 2), 128, 512, 0), (1, (34, 22, 20), (2, 2, 4), 128, 64, 0)])
def test_gemm_over_voxels_adds_stage_by_stage(n, dhw, grid, cin, cout, flat):
    family, (_, _, splits, staged) = route(sp3d.SP_OP_WGRAD, sp3d.Geom(n, dhw, grid, 1, 0, flat), cin, cout, sp3d.SP_BF16)
    assert family == "gemm" and staged and n * dhw[0] * dhw[1] * dhw[2] <= 36 * 64 * splits
    dw, db = weight_gradient(n, dhw, grid, cin, cout, "bf16", flat)
    assert dw <= chain(36 + 8), dw
    assert db <= 2.0 ** -24, db


# fp32: 16 voxels at a time; a workgroup has at most 16 bricks of 256 voxels, a quarter each for its waves: 64 sums of 16 in a
# chain, 4 waves, 512 workgroups in 16 runs: chain(16 + 64 + 4 + 32 + 16), and 15 % for the scatter of a norm over 216 values
# (three times 1 / sqrt(2 * 216)).  (Running sums over all voxels: 8.8e-7, 6.1e-7.)
@pytest.mark.parametrize("n, dhw, grid, cin, cout", [(1, (132, 112, 115), (1, 4, 1), 1, 8), (2, (132, 80, 114), (4, 4, 2), 8, 16)])
def test_fp32_weight_gradient_adds_sixteen_voxels_at_a_time(n, dhw, grid, cin, cout):
    dw, _ = weight_gradient(n, dhw, grid, cin, cout, "f32", 0)
    assert dw <= 1.15 * chain(132), dw


# bf16, 2 ... 8 channels: a wave's running sum of 32 products per row of a brick (rounded eight times each), four waves, and the
# workgroups in 16 runs; every case has at most 3 bricks per workgroup: chain(3 * 4 * 8 + 4 + 48 + 16).
@pytest.mark.parametrize("n, dhw, grid, cin, cout, flat", [
    (1, (41, 90, 163), (1, 2, 1), 3, 32, 0), (2, (33, 50, 97), (1, 1, 1), 4, 64, 0), (1, (30, 77, 130), (2, 1, 2), 7, 32, 0),
    (1, (33, 64, 96), (1, 1, 1), 8, 32, 0), (5, (2, 200, 258), (1, 2, 2), 5, 32, 1), (3, (4, 130, 95), (1, 1, 1), 2, 32, 1)])
def test_few_channel_weight_gradient(n, dhw, grid, cin, cout, flat):
    dw, db = weight_gradient(n, dhw, grid, cin, cout, "bf16", flat)
    assert dw <= chain(164) and db <= chain(164), (dw, db)


# 2-D, whole patches: eight waves of a workgroup add 16 products of a row to a running sum at a time (four roundings each), at most
# eight units of four rows each in these layers; then the waves and the workgroups: chain(8 * 4 * 4 + 8 + 40).  One unit, an
# odd number of them (half of a workgroup has nothing in its last step), more workgroups than steps, several steps.
@pytest.mark.parametrize("n, dhw, grid, cin, cout", [
    (1, (1, 8, 32), (1, 1, 1), 32, 32), (1, (3, 8, 32), (1, 1, 1), 64, 32), (1, (5, 24, 96), (1, 1, 1), 96, 64),
    (3, (7, 16, 64), (1, 2, 2), 32, 64), (1, (16, 128, 128), (1, 2, 2), 64, 128)])
def test_flat_whole_patches(n, dhw, grid, cin, cout):
    dw, db = weight_gradient(n, dhw, grid, cin, cout, "bf16", 1)
    assert dw <= chain(176) and db <= chain(176), (dw, db)
