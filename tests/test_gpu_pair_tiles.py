"""GPU parity of the pair buffer's tile sizes and rounds against the oracle, bit-exact.

C of every tile size (2^11 .. 2^14 entries a tile) and of one entry more and less than a whole number
of tiles, with few sorting workgroups and enough updates that some sort several rounds of them, and
with an output at an address that rules out the tile pass's 16-byte accesses.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M", [(2048, 1), (2049, 1), (683, 3), (40_000, 25), (50_001, 30), (33_000, 100), (70_001, 64)])
def test_tiles_and_rounds(fc, N, M):
    rng = np.random.default_rng(N + M)
    X, Y, Z = 48, 48, 48
    n = X * Y * Z
    roi = rng.integers(0, N, n).astype(np.int32).reshape(Z, Y, X)
    lab = np.where(rng.random(n) < 0.4, rng.integers(0, M, n), -1).astype(np.int32).reshape(Z, Y, X)
    S = 20_000
    lens = rng.integers(0, 16, S)
    off = np.zeros(S + 1, np.int64)
    off[1:] = np.cumsum(lens)
    pts = rng.uniform(-1, 48, (int(off[-1]), 3)).astype(np.float32)
    exp = oracle.count(pts, off, roi, lab, N, M)
    assert exp.sum() > (16 * 16384 * 1.2 if M > 20 else 20_000)
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, roi, lab)]
    for cap, shift in ((1 << 22, 0), (1 << 22, 1), (4096 * 8, 0)):
        print(f"pair tiles N={N} M={M} cap={cap} shift={shift}", flush=True)
        buf = torch.full((N * M + 1,), 5, dtype=torch.int32, device="cuda")
        out = buf[shift:shift + N * M].view(N, M)
        for acc in (False, True):
            fc.count(*dev, N, M, variant=2, blocks_per_cu=1, pair_capacity=cap, out=out, accumulate=acc)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), 2 * exp)
