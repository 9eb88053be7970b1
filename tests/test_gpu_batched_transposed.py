"""GPU parity of a plan that counts into transposed copies of C, bit-exact.

Plans of more than 2^24 points give every subject with a C of its own (N >= 64, M >= 2) such a copy.  One large
cheap subject, most of whose points lie outside its grid, takes this plan over that line; beside it subjects
of every kind (pass-through, both endpoint modes, seed to end, upsampled by 2 to 4), a C shared by two, ragged
N and M, M = 1 and N < 64 (no copies), and streamlines that outgrow the kernel's candidate lists, whose rows
and labels the fallback adds in the copies' layout.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_09247_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (50, 30, 20)


def _volumes(N, M, seed):
    rng = np.random.default_rng(seed)
    n = DIMS[0] * DIMS[1] * DIMS[2]
    roi = np.where(rng.random(n) < 0.5, rng.integers(0, N, n), -1).astype(np.int32)
    lab = np.where(rng.random(n) < 0.5, rng.integers(0, M, n), -1).astype(np.int32)
    return roi.reshape(DIMS[::-1]), lab.reshape(DIMS[::-1])


def _lines(S, seed, longest=12, step=1.0):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, longest, S)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    P = int(off[-1])
    start = np.repeat(rng.uniform(0, 1, (P // 8 + 1, 3)), 8, axis=0)[:P] * (np.array(DIMS) + 2) - 1
    return (start + step * rng.uniform(-1, 1, (P, 3))).astype(np.float32), off


def _large(S, per):
    """S streamlines of `per` points, all outside the grid but one in 400."""
    pts = torch.full((S * per, 3), 1000.0, dtype=torch.float32)
    g = torch.Generator().manual_seed(7)
    inside = torch.rand((S * per + 399) // 400, 3, generator=g) * torch.tensor(DIMS)
    pts[::400] = inside
    return pts.numpy(), np.arange(S + 1, dtype=np.int64) * per


SPECS = [  # N, M, mode, upsample, streamlines, longest, scale
    (4001, 13, 0, 1, 20_000, 12, 1.0), (65, 2, 1, 1, 5000, 12, 1.0), (700, 129, 2, 1, 5000, 12, 0.9),
    (1000, 64, 3, 1, 5000, 12, 1.0), (333, 70, 0, 2, 3000, 12, 1.0), (64, 31, 0, 3, 3000, 12, 1.1),
    (4097, 65, 0, 4, 3000, 12, 1.0), (500, 1, 0, 1, 3000, 12, 1.0), (63, 20, 0, 1, 3000, 12, 1.0),
    (20_000, 90, 0, 1, 60, 2500, 1.0), (20_000, 90, 2, 1, 60, 2500, 1.0), (20_000, 90, 0, 2, 60, 1500, 1.0),
]


def _subjects():
    subs = []
    for k, (N, M, mode, up, S, longest, scale) in enumerate(SPECS):
        roi, lab = _volumes(N, M, 40 + k)
        pts, off = _lines(S, 80 + k, longest, 20.0 if longest > 100 else 1.0)
        subs.append(dict(pts=pts, off=off, r=roi, l=lab, N=N, M=M, mode=mode, upsample=up, scale=scale))
    pts, off = _large(20_000, 845)   # 16.9M points
    roi, lab = _volumes(6000, 41, 1)
    subs.append(dict(pts=pts, off=off, r=roi, l=lab, N=6000, M=41, mode=0, upsample=1, scale=1.0))
    for seed in (300, 301):          # one C for both
        pts, off = _lines(4000, seed)
        subs.append(dict(pts=pts, off=off, r=subs[0]["r"], l=subs[0]["l"], N=4001, M=13, mode=0, upsample=1, scale=1.0, shared=True))
    shared = torch.empty((4001, 13), dtype=torch.int32, device="cuda")
    for s in subs:
        s["expect"] = oracle.count(s["pts"], s["off"], s["r"], s["l"], s["N"], s["M"], scale=s["scale"], mode=s["mode"],
                                   upsample=s["upsample"])
        assert s["expect"].sum() > 50, (s["N"], s["M"], s["mode"])
        s.update(points=torch.from_numpy(s["pts"]).cuda(), offsets=torch.from_numpy(s["off"]).cuda(),
                 roi=torch.from_numpy(s["r"]).cuda(), lab=torch.from_numpy(s["l"]).cuda(),
                 C=shared if s.get("shared") else torch.empty((s["N"], s["M"]), dtype=torch.int32, device="cuda"))
    subs[-1]["expect"] = subs[-2]["expect"] = subs[-1]["expect"] + subs[-2]["expect"]
    return subs


def test_transposed_copies_of_every_kind(fc):
    subs = _subjects()
    keys = ("points", "offsets", "roi", "lab", "N", "M", "mode", "upsample", "scale", "C")
    large = next(s for s in subs if s["N"] == 6000)
    # a plan of half the large subject's points takes no copies: less memory by at least them
    torch.cuda.synchronize()
    half = [dict({k: s[k] for k in keys}, **({"offsets": s["offsets"][:10_001].contiguous()} if s is large else {})) for s in subs]
    free0 = torch.cuda.mem_get_info()[0]
    small = fc.Plan(half)
    free1 = torch.cuda.mem_get_info()[0]
    small.close()
    free2 = torch.cuda.mem_get_info()[0]
    plan = fc.Plan([{k: s[k] for k in keys} for s in subs])
    free3 = torch.cuda.mem_get_info()[0]
    copies = sum(4 * s["N"] * s["M"] for s in subs if s["N"] >= 64 and s["M"] > 1 and not s.get("shared"))
    print(f"transposed plan: {sum(len(s['pts']) for s in subs)} points, copies {copies} bytes, plans {free0 - free1} "
          f"and {free2 - free3}", flush=True)
    assert (free2 - free3) - (free0 - free1) > copies - (4 << 20)
    for rep in range(3):
        for s in subs:
            s["C"].fill_(5 + rep)
        plan.launch()
        torch.cuda.synchronize()
        for k, s in enumerate(subs):
            np.testing.assert_array_equal(s["C"].cpu().numpy().astype(np.int64), s["expect"],
                                          err_msg=f"subject {k} (N={s['N']} M={s['M']} mode={s['mode']} u={s['upsample']}) launch {rep}")
    plan.close()
