"""GPU parity of the ranges that the flat-stream kernel's wavefronts find for themselves, bit-exact.

With one workgroup per CU of 256 CUs, 1024 wavefronts: ranges of equally many streamlines up to 2048, of about
equally many points and streamlines up to 32,768, and a table beyond.  Both sides of each line, with
streamlines in any order of length, giant ones, runs of empty ones, also at the ends, and only empty ones.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_09247_amd import synth

pytestmark = pytest.mark.gpu


def _lines(S, order, seed):
    rng = np.random.default_rng(seed)
    lens = np.clip(np.round(8 * np.exp(0.7 * rng.standard_normal(S))), 1, 60).astype(np.int64)
    if order == "falling":
        lens = np.sort(lens)[::-1].copy()
    if order == "long in a row":
        lens[: S // 20] *= 10
    if order == "empty runs":
        lens[: S // 4] = 0
        lens[S - S // 4:] = 0
        lens[rng.random(S) < 0.3] = 0
    if order == "giant":
        lens[S // 2] = 50_000
        lens[S - 1] = 20_000
    off = np.zeros(S + 1, np.int64)
    off[1:] = np.cumsum(lens)
    P = int(off[-1])
    base = np.repeat(rng.uniform(4, 60, (P // 16 + 1, 3)), 16, axis=0)[:P]
    return (base + rng.uniform(-2, 2, (P, 3))).astype(np.float32), off


@pytest.mark.parametrize("order", ["drawn", "falling", "long in a row", "empty runs", "giant"])
@pytest.mark.parametrize("waves", [2, 32])
@pytest.mark.parametrize("more", [0, 1])
def test_lines(fc, order, waves, more):
    vols = synth.volumes_interleaved64()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S = 4 * cus * waves + more
    pts, off = _lines(S, order, waves + more)
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, vols.roi, vols.lab)]
    vol = fc.Volume(dev[2], dev[3], vols.N, vols.M)
    for mode, up in ((0, 1), (2, 1), (0, 2)):
        exp = oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M, mode=mode, upsample=up)
        assert exp.sum() > 100
        print(f"own ranges S={S} {order} mode={mode} up={up}", flush=True)
        for kw in (dict(blocks_per_cu=1), dict(), dict(blocks_per_cu=1, batch=4)):
            C = fc.count(*dev, vols.N, vols.M, mode=mode, upsample=up, variant=2, **kw)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(C.cpu().numpy().astype(np.int64), exp, err_msg=f"{kw}")
        out = torch.full((vols.N, vols.M), 7, dtype=torch.int32, device="cuda")
        vol.count(dev[0], dev[1], mode=mode, upsample=up, out=out, noalloc=True, blocks_per_cu=1)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), exp, err_msg="noalloc")


def test_only_empty_streamlines(fc):
    vols = synth.volumes_interleaved64()
    dev = [torch.from_numpy(a).cuda() for a in (np.zeros((1, 3), np.float32), np.zeros(20_001, np.int64), vols.roi, vols.lab)]
    C = fc.count(*dev, vols.N, vols.M, variant=2, blocks_per_cu=1)
    torch.cuda.synchronize()
    assert not C.any()
