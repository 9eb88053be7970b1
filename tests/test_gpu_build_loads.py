"""GPU parity of the compact build's cached and non-temporal loads against the oracle, bit-exact: a grid of more
than 2^23 voxels, counted with one streamline less than 2^22 and with 2^22 (from there on the volumes are read
past the caches), rows of a length that no load divides, volumes at an odd 4-byte address.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def test_large_grid_on_either_side_of_the_line(fc):
    X, Y, Z = 203, 205, 207
    rng = np.random.default_rng(9)
    n = X * Y * Z
    assert n > 1 << 23
    N, M = 300, 9
    roi = np.where(rng.random(n) < 0.3, rng.integers(-2, N + 2, n), -1).astype(np.int32)
    lab = np.where(rng.random(n) < 0.3, rng.integers(-2, M + 2, n), -1).astype(np.int32)
    S = 1 << 22
    lens = rng.integers(1, 3, S)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    v = rng.permutation(n)
    v = np.concatenate([v, v])[: int(off[-1])]
    pts = np.stack([v % X, v // X % Y, v // (X * Y)], -1).astype(np.float32)
    buf = torch.empty(2 * n + 1, dtype=torch.int32, device="cuda")
    droi, dlab = buf[1:n + 1].view(Z, Y, X), buf[n + 1:].view(Z, Y, X)
    droi.copy_(torch.from_numpy(roi).view(Z, Y, X))
    dlab.copy_(torch.from_numpy(lab).view(Z, Y, X))
    dpts, doff = torch.from_numpy(pts).cuda(), torch.from_numpy(off).cuda()
    for s in (S - 1, S):
        exp = oracle.count(pts[: off[s]], off[: s + 1], roi.reshape(Z, Y, X), lab.reshape(Z, Y, X), N, M)
        assert exp.sum() > 100_000
        print(f"build loads S={s}", flush=True)
        got = fc.count(dpts, doff[: s + 1], droi, dlab, N, M, variant=2)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy().astype(np.int64), exp, err_msg=f"S={s}")
