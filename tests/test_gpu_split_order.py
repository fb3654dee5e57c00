"""The implicit GEMM with its K loop split between workgroups: which steps a split adds up, seen in the rounding of its sums."""
import numpy as np
import pytest
import torch

from gpu_util import DT, route
from paper_1909_03108_amd import sp3d

BF16 = DT["bf16"]
# n, dhw, cin, cout, 2-D, (output blocks per wave, tiles of 128 voxels, record loads, splits).  Every shape of the kernel, with splits that
# begin in the middle of three steps, with an item per workgroup and with several in a row.
LAYERS = [(1, (8, 8, 8), 128, 128, 0, (2, 1, 3, 9)), (2, (1, 1, 5), 96, 192, 0, (1, 1, 3, 6)), (1, (16, 16, 16), 256, 256, 0, None),
          (1, (4, 4, 4), 512, 512, 0, None), (2, (16, 16, 16), 512, 256, 1, None),
          (1, (1, 1, 2), 96, 192, 0, (1, 1, 4, 6)), (2, (1, 1, 1), 96, 192, 0, (1, 1, 6, 6)), (2, (2, 28, 33), 288, 192, 0, (1, 2, 5, 5)),
          (2, (76, 6, 4), 288, 192, 0, (1, 2, 6, 5)), (1, (1, 1, 2), 96, 128, 0, (2, 1, 4, 6)), (1, (1, 1, 1), 96, 128, 0, (2, 1, 6, 6)),
          (1, (9, 69, 18), 288, 128, 0, (2, 2, 5, 5)), (1, (60, 30, 7), 384, 128, 0, (2, 2, 6, 5)),
          (2, (7, 17, 62), 608, 192, 0, (1, 1, 3, 2)), (2, (79, 31, 3), 608, 192, 0, (1, 1, 4, 2)),
          (2, (32, 69, 1), 992, 320, 0, (1, 1, 6, 5)), (2, (3, 46, 79), 704, 128, 0, (2, 1, 3, 4)),
          (2, (75, 80, 2), 800, 128, 0, (2, 1, 4, 4)), (2, (59, 66, 1), 736, 384, 0, (2, 1, 6, 4)),
          (2, (89, 5, 28), 832, 128, 0, (2, 2, 5, 5)), (2, (45, 58, 5), 832, 128, 0, (2, 2, 6, 5))]


@pytest.mark.gpu
@pytest.mark.parametrize("n, dhw, cin, cout, flat, cut", LAYERS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_a_split_adds_its_share_of_the_steps_in_order(n, dhw, cin, cout, flat, cut):
    """A step is a kernel row times 32 input channels, chunks innermost; split s has the steps [s nk / S, (s + 1) nk / S), and the
    splits' sums are added in order, the bias before the first split's first step.  One product of a step is not zero: 2^40 in one step of each output channel, -2^40 in another,
    1 in the others, so that what is added between the two, and only that, is lost: every cut of the steps has its own integers."""
    g = sp3d.Geom(n, dhw, (1, 1, 1), flat=flat)
    kind, detail = route(sp3d.SP_OP_FWD, g, cin, cout, BF16)
    splits = detail[3]
    assert kind == "gemm" and splits > 1 and (cut is None or detail == cut), (kind, detail)
    nci, nrows = cin // 32, 3 if flat else 9
    nk = nci * nrows
    rng = np.random.default_rng(17)
    big = np.argsort(rng.random((cout, nk)), axis=1)[:, :2]              # two different steps per output channel
    p = np.ones((cout, nk), np.float32)
    p[np.arange(cout), big[:, 0]] = 2.0 ** 40
    p[np.arange(cout), big[:, 1]] = -(2.0 ** 40)
    chan = 32 * np.arange(nci) + rng.integers(0, 32, nci)                # the channel of a chunk that is not zero
    w = np.zeros((3, 3, 3, cin, cout) if not flat else (1, 3, 3, cin, cout), np.float32)
    x = torch.zeros((n,) + dhw + (cin,), dtype=torch.bfloat16, device="cuda")
    x[..., torch.from_numpy(chan).cuda()] = 1.0
    D, H, W = dhw
    # [row][d][h]: does the row of the kernel lie in the volume
    inside = np.zeros((nrows, D, H), bool)
    for r in range(nrows):
        kd, kh = (0, r) if flat else (r // 3, r % 3)
        w[kd, kh, 1, chan] = p[:, r * nci:(r + 1) * nci].T
        dd = np.arange(D) + (0 if flat else kd - 1)
        hh = np.arange(H) + kh - 1
        inside[r] = ((dd >= 0) & (dd < D))[:, None] & ((hh >= 0) & (hh < H))[None, :]
    bias = rng.integers(0, 8, cout).astype(np.float32)
    want = np.zeros((D, H, cout), np.float32)
    for s in range(splits):
        part = np.zeros((D, H, cout), np.float32) + (bias if s == 0 else 0)
        for k in range(s * nk // splits, (s + 1) * nk // splits):
            part += inside[k // nci][..., None] * p[:, k]
        want += part
    want = torch.from_numpy(want).to(torch.bfloat16).cuda()
    P, Py = sp3d.alloc_padded(g, cin, BF16), sp3d.alloc_padded(g, cout, BF16)
    sp3d.sp_partition(x, P, g, cin, BF16)
    wd = torch.from_numpy(w if not flat else w[0]).to(torch.bfloat16).cuda()
    ws = sp3d.alloc_ws(sp3d.sp_workspace_bytes(sp3d.SP_OP_FWD, g, cin, cout, BF16))
    sp3d.conv3d_fwd(P, wd, torch.from_numpy(bias).cuda(), Py, g, cin, cout, BF16, 0, ws)
    y = torch.empty((n,) + dhw + (cout,), dtype=torch.bfloat16, device="cuda")
    sp3d.sp_unpartition(Py, y, g, cout, BF16)
    wrong = (y != want[None, :, :, None, :]).sum().item()
    assert wrong == 0, "%d of %d sums" % (wrong, y.numel())
