"""GPU parity of the one-pass compact volume build against the oracle, bit-exact.

Every voxel of a grid whose sizes straddle the build's units (4-voxel loads, 16x8x8 super-bricks,
64-voxel wavefronts along x) is a point of some streamline, so a wrong bit, base or code shows.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (1, 9, 9), (2, 5, 3), (3, 8, 2), (4, 4, 4), (5, 7, 9), (15, 8, 8), (16, 16, 16), (17, 9, 17),
        (63, 3, 5), (64, 8, 8), (65, 9, 10), (67, 2, 33), (130, 17, 7), (256, 3, 3), (259, 5, 2)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("fill", [0.03, 0.4, 1.0])
def test_every_voxel(fc, dims, fill):
    X, Y, Z = dims
    rng = np.random.default_rng(X + 1000 * Y + int(100 * fill))
    N, M = 40, 7
    n = X * Y * Z
    # values outside [0, N) and [0, M) are no hits
    roi = np.where(rng.random(n) < fill, rng.integers(-3, N + 3, n), -1).astype(np.int32).reshape(Z, Y, X)
    lab = np.where(rng.random(n) < fill, rng.integers(-3, M + 3, n), -1).astype(np.int32).reshape(Z, Y, X)
    z, y, x = np.meshgrid(np.arange(Z), np.arange(Y), np.arange(X), indexing="ij")
    pts = np.stack([x, y, z], -1).reshape(-1, 3).astype(np.float32)
    pts = pts[rng.permutation(n)]
    off = np.append(np.arange(0, n, 9), n).astype(np.int64)
    exp = oracle.count(pts, off, roi, lab, N, M)
    print(f"compact dims={dims} fill={fill}", flush=True)
    # the volumes start at an odd 4-byte address
    buf = torch.empty(2 * n + 2, dtype=torch.int32, device="cuda")
    droi, dlab = buf[1:n + 1].view(Z, Y, X), buf[n + 1:2 * n + 1].view(Z, Y, X)
    droi.copy_(torch.from_numpy(roi))
    dlab.copy_(torch.from_numpy(lab))
    dpts, doff = torch.from_numpy(pts).cuda(), torch.from_numpy(off).cuda()
    got = fc.count(dpts, doff, droi, dlab, N, M, variant=2)
    vol = fc.Volume(droi, dlab, N, M)
    got2 = vol.count(dpts, doff)
    C = torch.empty((N, M), dtype=torch.int32, device="cuda")
    plan = fc.Plan([dict(points=dpts, offsets=doff, roi=droi, lab=dlab, N=N, M=M, C=C)])
    plan.launch()
    torch.cuda.synchronize()
    for name, g in (("plain", got), ("resident", got2), ("plan", C)):
        np.testing.assert_array_equal(g.cpu().numpy().astype(np.int64), exp, err_msg=name)
