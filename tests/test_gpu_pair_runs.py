"""GPU parity of the pair histogram where most updates fall into one tile of C, bit-exact.

The tile pass takes runs of 72 updates or more 64 at a time from a 16-byte boundary: hot tiles of every tile
size, first, last (also a partial one) or between others, whose other updates shift the runs' starts; a
single hot entry; few and many sorting workgroups, and runs of several rounds.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

X = Y = Z = 40


@pytest.mark.parametrize("N,M", [(500, 4), (2048, 1), (683, 3), (40_000, 25), (50_001, 30), (33_000, 100), (70_001, 64)])
@pytest.mark.parametrize("hot", ["first", "last", "middle", "one entry"])
def test_hot_tile(fc, N, M, hot):
    rng = np.random.default_rng(N + M + len(hot))
    n = X * Y * Z
    rows = {"first": 12, "last": 12, "middle": 12, "one entry": 1}[hot]
    lo = {"first": 0, "last": N - rows, "middle": (N - rows) // 2, "one entry": N // 3}[hot]
    roi = np.where(rng.random(n) < 0.9, lo + rng.integers(0, rows, n), rng.integers(0, N, n))
    lab = np.where(rng.random(n) < 0.9, rng.integers(0, 1 if rows == 1 else min(M, 3), n), rng.integers(0, M, n))
    lab[rng.random(n) < 0.3] = -1
    roi, lab = (a.astype(np.int32).reshape(Z, Y, X) for a in (roi, lab))
    S = 24_000
    lens = rng.integers(0, 9, S)
    off = np.zeros(S + 1, np.int64)
    off[1:] = np.cumsum(lens)
    pts = rng.uniform(-1, X, (int(off[-1]), 3)).astype(np.float32)
    exp = oracle.count(pts, off, roi, lab, N, M)
    assert exp.max() > 500
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, roi, lab)]
    for kw in (dict(blocks_per_cu=1), dict()):
        print(f"pair runs N={N} M={M} hot={hot} {kw}", flush=True)
        out = torch.full((N, M), 5, dtype=torch.int32, device="cuda")
        for acc in (False, True):
            fc.count(*dev, N, M, variant=2, pair_capacity=1 << 22, out=out, accumulate=acc, **kw)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), 2 * exp)
