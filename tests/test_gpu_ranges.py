"""GPU parity of the flat-stream kernel's streamline ranges against the oracle, bit-exact.

Up to four streamlines per wavefront of a full launch, every wavefront gets one range of (nearly)
equally many streamlines; beyond that, ranges come from a table written in one pass over the offsets.
Both sides of that line, calls smaller than one workgroup, streamlines long enough to begin hundreds
of ranges at once, and runs of empty streamlines, also at the ends.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_09247_amd import synth

pytestmark = pytest.mark.gpu


def _case(S, giant, seed):
    vols = synth.volumes_interleaved64()
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 9, S)
    lens[rng.random(S) < 0.2] = 0
    lens[: S // 8] = 0
    lens[S - S // 8:] = 0
    if giant:
        lens[S // 2] = 60 * max(S, 50)
    off = np.zeros(S + 1, np.int64)
    off[1:] = np.cumsum(lens)
    P = int(off[-1])
    # points near the middle of the grid, in runs that stay close to each other
    base = np.repeat(rng.uniform(4, 60, (P // 16 + 1, 3)), 16, axis=0)[:P]
    pts = (base + rng.uniform(-2, 2, (P, 3))).astype(np.float32).reshape(-1, 3)
    return pts, off, vols


@pytest.mark.parametrize("S", [1, 3, 5, 1023, 1025, 4096, 4097, 9001])
@pytest.mark.parametrize("giant", [False, True])
def test_ranges(fc, S, giant):
    pts, off, vols = _case(S, giant, 100 + S)
    if pts.shape[0] == 0:
        pts = np.zeros((1, 3), np.float32)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, vols.roi, vols.lab)]
    vol = fc.Volume(dev[2], dev[3], vols.N, vols.M)
    for mode in (0, 2):
        exp = oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M, mode=mode)
        # one workgroup per CU: with 256 CUs the line lies at 4 * 4 * 256 = 4096 streamlines
        print(f"ranges S={S} giant={giant} mode={mode} cus={cus}", flush=True)
        for kw in (dict(blocks_per_cu=1), dict()):
            C = fc.count(*dev, vols.N, vols.M, mode=mode, variant=2, **kw)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(C.cpu().numpy().astype(np.int64), exp, err_msg=f"{kw}")
        out = torch.full((vols.N, vols.M), 7, dtype=torch.int32, device="cuda")
        vol.count(dev[0], dev[1], mode=mode, out=out, noalloc=True, blocks_per_cu=1)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), exp, err_msg="noalloc")


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("batch", [2, 4])
def test_end_labels_at_window_edges(fc, mode, batch):
    # streamlines whose ends lie on either side of the kernel's 64-point windows and of its batches,
    # with stretches without any hit between hits (windows and batches that look nothing up)
    vols = synth.volumes_interleaved64()
    rng = np.random.default_rng(7 * mode + batch)
    lens = rng.choice([0, 1, 2, 62, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257], 3000)
    off = np.zeros(lens.size + 1, np.int64)
    off[1:] = np.cumsum(lens)
    P = int(off[-1])
    pts = (np.repeat(rng.uniform(4, 60, (P // 8 + 1, 3)), 8, axis=0)[:P] + rng.uniform(-2, 2, (P, 3))).astype(np.float32)
    far = np.repeat(rng.random(P // 48 + 1) < 0.6, 48)[:P]
    pts[far] += 1000.0
    ends = np.concatenate([off[:-1][lens > 0], off[1:][lens > 0] - 1])
    pts[ends] = np.where(far[ends, None], pts[ends] - 1000.0, pts[ends])   # most ends do hit
    exp = oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M, mode=mode)
    assert exp.sum() > 1000
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, vols.roi, vols.lab)]
    for kw in (dict(blocks_per_cu=1), dict()):
        print(f"end labels mode={mode} batch={batch} {kw}", flush=True)
        C = fc.count(*dev, vols.N, vols.M, mode=mode, variant=2, batch=batch, **kw)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(C.cpu().numpy().astype(np.int64), exp, err_msg=f"{kw}")


@pytest.mark.parametrize("sizes", [(1, 1, 1), (3, 4097, 0, 70), (20_000, 30_000), (150_000, 5)])
def test_batched_items(fc, sizes):
    # plans with fewer work items than wavefronts and with more, streamlines that begin hundreds of
    # items, runs of empty ones, a subject without streamlines
    subs, exps = [], []
    for k, S in enumerate(sizes):
        pts, off, vols = _case(max(S, 1), k % 2 == 1, 300 + k)
        off = off[: S + 1]
        pts = pts[: int(off[-1])]
        exps.append(oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M))
        pts = pts if len(pts) else np.zeros((1, 3), np.float32)   # (never read)
        subs.append(dict(points=torch.from_numpy(pts).cuda(), offsets=torch.from_numpy(off).cuda(),
                         roi=torch.from_numpy(vols.roi).cuda(), lab=torch.from_numpy(vols.lab).cuda(), N=vols.N, M=vols.M,
                         C=torch.empty((vols.N, vols.M), dtype=torch.int32, device="cuda")))
    print(f"batched items sizes={sizes} points={[s['points'].shape[0] for s in subs]}", flush=True)
    plan = fc.Plan(subs)
    for _ in range(3):
        for s in subs:
            s["C"].fill_(9)
        plan.launch()
        torch.cuda.synchronize()
        for k, s in enumerate(subs):
            np.testing.assert_array_equal(s["C"].cpu().numpy().astype(np.int64), exps[k], err_msg=f"subject {k}")


@pytest.mark.parametrize("S", [1, 62, 63, 64, 65, 126, 127, 5000])
def test_seed_end_lines(fc, S):
    # a wavefront counts 63 streamlines at a time; one-point and empty ones, also at the ends
    pts, off, vols = _case(S, False, 500 + S)
    off = np.concatenate([off[:1], off]) if S % 2 else off
    if off[-1] == 0:
        off[-1] = 1
    pts = pts[: int(off[-1])] if len(pts) >= off[-1] else np.full((int(off[-1]), 3), 20, np.float32)
    exp = oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M, mode=3)
    dev = [torch.from_numpy(a).cuda() for a in (pts, off, vols.roi, vols.lab)]
    print(f"seed end S={S}", flush=True)
    C = torch.empty((vols.N, vols.M), dtype=torch.int32, device="cuda")
    plan = fc.Plan([dict(points=dev[0], offsets=dev[1], roi=dev[2], lab=dev[3], N=vols.N, M=vols.M, C=C, mode=3)])
    plan.launch()
    for variant in (1, 2):
        got = fc.count(*dev, vols.N, vols.M, mode=3, variant=variant)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy().astype(np.int64), exp, err_msg=f"variant {variant}")
    np.testing.assert_array_equal(C.cpu().numpy().astype(np.int64), exp, err_msg="plan")
