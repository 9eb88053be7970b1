"""GPU parity of plans and served bursts whose subjects differ widely in size, bit-exact: one large subject
among hundreds of little ones (first, in between, last), a large C with few streamlines, subjects without
streamlines and of every kind.  Their preparation gives the large one workgroups in proportion.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_09247_amd import synth

pytestmark = pytest.mark.gpu


def _lines(S, seed, hi=9):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, hi, S)
    off = np.zeros(S + 1, np.int64)
    off[1:] = np.cumsum(lens)
    P = int(off[-1])
    base = np.repeat(rng.uniform(4, 60, (P // 16 + 1, 3)), 16, axis=0)[:P]
    return (base + rng.uniform(-2, 2, (P, 3))).astype(np.float32), off


@pytest.mark.parametrize("place", ["first", "middle", "last"])
@pytest.mark.parametrize("n", [40, 300])
def test_one_large_subject(fc, place, n):
    vols = synth.volumes_interleaved64()
    roi, lab = torch.from_numpy(vols.roi).cuda(), torch.from_numpy(vols.lab).cuda()
    at = {"first": 0, "middle": n // 2, "last": n - 1}[place]
    wide = np.arange(64 * 64 * 64, dtype=np.int32).reshape(64, 64, 64) % 200_000
    subs, exps, cache = [], [], {}
    for k in range(n):
        S = 150_000 if k == at else (0 if k % 11 == 3 else 20 + k % 7)
        mode, up = ((0, 1), (2, 1), (3, 1), (0, 2))[k % 4] if k != at else (0, 1)
        N, r = (200_000, wide) if k == 5 else (vols.N, vols.roi)
        key = (S, mode, up, k == 5)
        if key not in cache:
            pts, off = _lines(S, S + mode)
            cache[key] = (torch.from_numpy(pts if len(pts) else np.zeros((1, 3), np.float32)).cuda(), torch.from_numpy(off).cuda(),
                          oracle.count(pts, off, r, vols.lab, N, vols.M, mode=mode, upsample=up))
        p, o, exp = cache[key]
        exps.append(exp)
        subs.append(dict(points=p, offsets=o, roi=torch.from_numpy(r).cuda() if k == 5 else roi, lab=lab, N=N, M=vols.M, mode=mode,
                         upsample=up, C=torch.full((N, vols.M), 9, dtype=torch.int32, device="cuda")))
    assert exps[at].sum() > 10_000
    print(f"one large subject {place} of {n}", flush=True)
    plan = fc.Plan(subs)
    for rep in range(2):
        plan.launch()
        torch.cuda.synchronize()
        for k, s in enumerate(subs):
            np.testing.assert_array_equal(s["C"].cpu().numpy().astype(np.int64), exps[k], err_msg=f"subject {k} rep {rep}")
            s["C"].fill_(-4)
    plan.close()


def test_one_large_request(fc):
    vols = synth.volumes_interleaved64()
    srv = fc.Server(memory_budget=256 << 20)
    vid = srv.add_volume(torch.from_numpy(vols.roi), torch.from_numpy(vols.lab), vols.N, vols.M)
    reqs = []
    for k in range(60):
        S = 150_000 if k == 7 else 5 + k
        pts, off = _lines(S, 70 + k)
        out = torch.full((vols.N, vols.M), -1, dtype=torch.int32, pin_memory=True)
        mode = 3 if k % 5 == 1 else 0
        reqs.append((torch.from_numpy(pts if len(pts) else np.zeros((1, 3), np.float32)).cuda(), torch.from_numpy(off), out,
                     oracle.count(pts, off, vols.roi, vols.lab, vols.N, vols.M, mode=mode), mode))
    torch.cuda.synchronize()
    print("one large request of 60", flush=True)
    for rep in range(2):
        ids = [srv.submit(vid, p, o, out, mode=mode) for p, o, out, _, mode in reqs]
        for rid, (_, _, out, exp, _) in zip(ids, reqs):
            assert srv.wait(rid)["status"] == fc.OK
        for k, (_, _, out, exp, _) in enumerate(reqs):
            np.testing.assert_array_equal(out.numpy().astype(np.int64), exp, err_msg=f"request {k} rep {rep}")
            out.fill_(-1)
    srv.close()
