"""Workloads by which this framework's speed is judged, through its public entry points.

Every case is one pass of one of the calls a program makes: a plain count (volumes and streamlines in
device memory), counts against a resident volume (one call, or a tractogram that arrives in pieces),
one launch of a batched plan, a burst of requests to the server, and the parcellation of a finished
matrix.  Inputs follow the recipe of the repository's synthetic subjects: an ellipsoidal brain mask
proportional to the grid, a bilateral seed ROI whose voxels are the rows of C in raster order, M labels
tiling a 3-voxel shell, and walks of 0.5-voxel steps that stop at the mask.

listed() are the cases, draw(rng) gives one more of the same ranges, prepare/run/work/exact as below.
"""
import functools
import math

import numpy as np
import torch

from paper_2302_09247_amd import fastcod, synth

SR = synth.SR_SCALE
DIMS_125 = (145, 174, 145)      # a 1.25 mm grid
DIMS_07 = (260, 311, 260)       # a 0.7 mm grid


def listed():
    return [
        # the smallest plain call: a 64^3 grid, ten thousand short walks; launches and latency count
        dict(name="plain_64", form="count", X=64, Y=64, Z=64, rows=2300, M=8, S=10_000, median=90, hi=200),
        # a selected bundle against a subject that is already on the device (interactive use)
        dict(name="bundle_resident", form="resident", X=145, Y=174, Z=145, rows=8000, M=70, S=1_000, median=150, hi=600),
        # a tractogram read from file in pieces, counted into one matrix without allocating; odd sizes
        dict(name="pieces_noalloc", form="noalloc", X=91, Y=109, Z=91, rows=5200, M=68, S=20_011, median=97, hi=411, pieces=5),
        # a whole 1.25 mm subject, one plain call
        dict(name="plain_125", form="count", X=145, Y=174, Z=145, rows=8000, M=70, S=1_000_000, median=150, hi=600),
        # the largest: a whole 0.7 mm subject of five million streamlines, one plain call
        dict(name="plain_07", form="count", X=260, Y=311, Z=260, rows=45_800, M=180, S=5_000_000, median=270, hi=1000),
        # labels of both ends only, against the resident 0.7 mm subject
        dict(name="ends_07", form="resident", X=260, Y=311, Z=260, rows=45_800, M=180, S=400_000, median=270, hi=1000, mode=2),
        # super-resolution: 1.25 mm walks on the 0.7 mm volumes, one point inserted between neighbours
        dict(name="superres_u2", form="resident", X=260, Y=311, Z=260, rows=45_800, M=180, S=300_000, median=150, hi=600, scale=SR, up=2),
        # Alg. 1's seed-to-end count of a 1.25 mm subject
        dict(name="seed_end_125", form="resident", X=145, Y=174, Z=145, rows=8000, M=70, S=1_000_000, median=150, hi=600, mode=3),
        # a study: subjects of uneven grids, ROI sizes, label counts and streamlines in one plan
        dict(name="study_batched", form="batched", subjects=12, X=145, Y=174, Z=145, rows=40_000, M=360, S=300_000, median=150, hi=600),
        # the same in small: many little subjects, where the plan's launches and item starts count
        dict(name="little_batched", form="batched", subjects=24, X=80, Y=97, Z=80, rows=3000, M=70, S=3000, median=80, hi=300),
        # a burst of requests to the server, device-resident streamlines, matrices to pinned host memory
        dict(name="burst_served", form="served", subjects=12, X=145, Y=174, Z=145, rows=8000, M=70, S=200_000, median=150, hi=600),
        # parcellation outputs of a 0.7 mm subject's matrix
        dict(name="parcellate_07", form="parcellate", rows=45_808, M=180, density=0.08),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choices(["count", "resident", "noalloc", "batched", "served", "parcellate"], [6, 6, 2, 3, 2, 2])[0]
    if form == "parcellate":
        return dict(form=form, rows=_log(rng, 900, 60_000), M=_log(rng, 2, 400), density=round(rng.uniform(0.02, 0.6), 3))
    c = dict(form=form, X=_log(rng, 48, 260), Y=_log(rng, 48, 311), Z=_log(rng, 48, 260), M=_log(rng, 4, 360),
             median=_log(rng, 40, 270))
    c["rows"] = min(_log(rng, 1000, 46_000), c["X"] * c["Y"] * c["Z"] // 40)
    c["hi"] = int(c["median"] * rng.uniform(2.0, 4.0))
    if form in ("batched", "served"):
        for k in "XYZ":
            c[k] = min(c[k], 174)
        c["rows"] = min(c["rows"], c["X"] * c["Y"] * c["Z"] // 40)
        c["subjects"] = rng.randint(2, 24)
        c["S"] = _log(rng, 1000, 150_000)
        return c
    c["S"] = _log(rng, 400, 1_500_000)
    if form == "noalloc":
        c["pieces"] = rng.randint(1, 6)
    kind = rng.choices(["pass", "ends", "both", "seed", "up"], [8, 1, 1, 1, 2])[0]
    if kind in ("ends", "both", "seed"):
        c["mode"] = {"ends": 1, "both": 2, "seed": 3}[kind]
    if kind == "up":
        c["up"] = rng.randint(2, 4)
    if kind == "up" or rng.random() < 0.25:
        c["scale"] = rng.choice([SR, 1.25, 0.8, 1.5625])
    return c


# ---- inputs ----

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _ellipsoid(dims, centre, semi, dev):
    z, y, x = (torch.arange(n, dtype=torch.float64, device=dev) for n in (dims[2], dims[1], dims[0]))
    return (((x[None, None, :] - centre[0]) / semi[0]) ** 2 + ((y[None, :, None] - centre[1]) / semi[1]) ** 2
            + ((z[:, None, None] - centre[2]) / semi[2]) ** 2) <= 1.0


def _anatomy(dims, rows):
    """Centre, brain semi-axes, and the two ROI ellipsoids scaled to about `rows` voxels in all."""
    centre = tuple((d - 1) / 2.0 for d in dims)
    brain = tuple(d * b / g for d, b, g in zip(dims, synth.CFG2_BRAIN, synth.CFG2_DIMS))
    ratio = tuple(d / g for d, g in zip(dims, synth.CFG2_DIMS))
    base = 2 * 4.0 / 3.0 * math.pi * math.prod(synth.CFG2_ROI_SEMI) * math.prod(ratio)
    f = (rows / base) ** (1.0 / 3.0)
    semi = tuple(max(1.0, a * r * f) for a, r in zip(synth.CFG2_ROI_SEMI, ratio))
    at = [tuple(centre[i] + (rc[i] - synth.CFG2_CENTRE[i]) * ratio[i] for i in range(3)) for rc in synth.CFG2_ROI_CENTRES]
    return centre, brain, semi, at


def _volumes(dims, rows, M, g, dev):
    """ROI index and label volumes [Z,Y,X] int32 and N; the label centroids come from the generator."""
    centre, brain, semi, at = _anatomy(dims, rows)
    mask = _ellipsoid(dims, centre, brain, dev)
    shell = mask & ~_ellipsoid(dims, centre, tuple(max(0.5, a - 3.0) for a in brain), dev)
    inside = (_ellipsoid(dims, at[0], semi, dev) | _ellipsoid(dims, at[1], semi, dev)) & ~shell
    flat = inside.reshape(-1)
    N = int(flat.sum())
    roi = torch.where(flat, torch.cumsum(flat, 0) - 1, -1).to(torch.int32).reshape(mask.shape)
    zyx = torch.nonzero(shell).to(torch.int32)
    cent = zyx[torch.randperm(zyx.shape[0], generator=g, device=dev)[:M]]
    lab = torch.full(mask.shape, -1, dtype=torch.int32, device=dev)
    near = torch.cat([((v[:, None] - cent[None]) ** 2).sum(-1).argmin(1) for v in zyx.split(1 << 17)])
    lab[shell] = near.to(torch.int32)
    return roi, lab, N


def _walks(dims, rows, S, median, hi, scale, g, dev):
    """Points [P,3] float32 and offsets [S+1] int64: walks on the grid whose coordinates times `scale`
    are those of the volumes."""
    centre, brain, semi, at = _anatomy(dims, rows)
    centre, brain, semi, at = [tuple(v / scale for v in t) for t in (centre, brain, semi)] + [[tuple(v / scale for v in a) for a in at]]
    c = torch.tensor(centre, dtype=torch.float64, device=dev)
    b = torch.tensor(brain, dtype=torch.float64, device=dev)
    pts, lens = [], []
    for lo in range(0, S, synth.CHUNK):
        n = min(synth.CHUNK, S - lo)
        T = torch.randn(n, generator=g, device=dev, dtype=torch.float64)
        T = torch.clamp(torch.round(median * torch.exp(0.5 * T)), 20, hi).to(torch.int64)
        side = torch.rand(n, 1, generator=g, device=dev) < 0.5
        seed = torch.where(side, synth.uniform_in_ellipsoid(n, at[0], semi, g, dev), synth.uniform_in_ellipsoid(n, at[1], semi, g, dev))
        seed = torch.where(torch.rand(n, 1, generator=g, device=dev) < 0.4, seed, synth.uniform_in_ellipsoid(n, centre, brain, g, dev))
        p, k = synth.random_walks(n, seed, T, g, lambda q: (((q - c) / b) ** 2).sum(-1) <= 1.0)
        pts.append(p)
        lens.append(k)
    off = torch.zeros(S + 1, dtype=torch.int64, device=dev)
    off[1:] = torch.cumsum(torch.cat(lens), 0)
    return torch.cat(pts) if len(pts) > 1 else pts[0], off


def _generator(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1_000_003 + 12345)
    return g


def _subject(case, g, dev):
    dims = (case["X"], case["Y"], case["Z"])
    roi, lab, N = _volumes(dims, case["rows"], case["M"], g, dev)
    pts, off = _walks(dims, case["rows"], case["S"], case["median"], case["hi"], case.get("scale", 1.0), g, dev)
    return dict(points=pts, offsets=off, roi=roi, lab=lab, N=N, M=case["M"], scale=case.get("scale", 1.0),
                mode=case.get("mode", 0), up=case.get("up", 1))


def _shrunk(case, k):
    """Subject k of a batched or served case: every size between a third of the case's and all of it."""
    r = np.random.default_rng([k, case["X"], case["S"]])
    f = lambda v, lo: max(lo, int(round(v * r.uniform(0.34, 1.0))))   # noqa: E731
    c = dict(case, X=f(case["X"], 40), Y=f(case["Y"], 40), Z=f(case["Z"], 40), M=f(case["M"], 3), S=f(case["S"], 100))
    c["rows"] = min(f(case["rows"], 200), c["X"] * c["Y"] * c["Z"] // 40)
    return c


def _subjects(case, seed):
    dev = _device()
    g = _generator(seed, dev)
    if case["form"] in ("batched", "served"):
        return [_subject(_shrunk(case, k), g, dev) for k in range(case["subjects"])]
    return [_subject(case, g, dev)]


def _matrix(case, seed):
    """A count matrix as streamlines give it: few labels per row, a few large entries, some empty rows."""
    dev = _device()
    g = _generator(seed, dev)
    shape = (case["rows"], case["M"])
    C = torch.exp(1.5 * torch.randn(shape, generator=g, device=dev)).to(torch.int32)
    C *= torch.rand(shape, generator=g, device=dev) < case["density"]
    C[torch.rand(shape[0], generator=g, device=dev) < 0.02] = 0
    return C


def prepare(case, seed):
    form = case["form"]
    if form == "parcellate":
        return dict(form=form, C=_matrix(case, seed))
    subs = _subjects(case, seed)
    st = dict(form=form)
    if form == "count":
        st.update(subs[0])
        st["C"] = torch.empty((st["N"], st["M"]), dtype=torch.int32, device=st["points"].device)
    elif form in ("resident", "noalloc"):
        s = subs[0]
        st["vol"] = fastcod.Volume(s.pop("roi"), s.pop("lab"), s["N"], s["M"])
        st["opts"] = dict(scale=s["scale"], mode=s["mode"], upsample=s["up"])
        st["C"] = torch.empty((s["N"], s["M"]), dtype=torch.int32, device=s["points"].device)
        n = case.get("pieces", 1)
        cut = [case["S"] * k // n for k in range(n + 1)]
        st["pieces"] = []
        for a, b in zip(cut, cut[1:]):
            lo, hi = int(s["offsets"][a]), int(s["offsets"][b])
            st["pieces"].append((s["points"][lo:hi].clone(), (s["offsets"][a:b + 1] - lo).contiguous()))
    elif form == "batched":
        for s in subs:
            s["C"] = torch.empty((s["N"], s["M"]), dtype=torch.int32, device=s["points"].device)
        st["plan"] = fastcod.Plan(subs)
        st["C"] = [s["C"] for s in subs]
    elif form == "served":
        room = sum(48 * s["roi"].numel() // 4 + 9 * s["offsets"].numel() + 4 * s["N"] * s["M"] for s in subs) + (64 << 20)
        st["server"] = fastcod.Server(memory_budget=room)
        st["requests"] = []
        for s in subs:
            vid = st["server"].add_volume(s["roi"].cpu(), s["lab"].cpu(), s["N"], s["M"])
            out = torch.empty((s["N"], s["M"]), dtype=torch.int32, pin_memory=True)
            st["requests"].append((vid, s["points"], s["offsets"].cpu(), out))
    return st


def run(st):
    form = st["form"]
    if form == "count":
        return fastcod.count(st["points"], st["offsets"], st["roi"], st["lab"], st["N"], st["M"], scale=st["scale"],
                             upsample=st["up"], mode=st["mode"], out=st["C"])
    if form in ("resident", "noalloc"):
        for k, (points, offsets) in enumerate(st["pieces"]):
            st["vol"].count(points, offsets, out=st["C"], accumulate=k > 0, noalloc=form == "noalloc", **st["opts"])
        return st["C"]
    if form == "batched":
        st["plan"].launch()
        return st["C"]
    if form == "served":
        ids = [st["server"].submit(vid, points, offsets, out) for vid, points, offsets, out in st["requests"]]
        for rid in ids:
            if st["server"].wait(rid)["status"] != fastcod.OK:
                raise RuntimeError("a request failed")
        return [r[3] for r in st["requests"]]
    lab, frac, sums = fastcod.parcellate(st["C"])
    return {"label": lab, "fractions": frac, "sums": sums}


# ---- the work a pass cannot do without ----

@functools.lru_cache(maxsize=None)
def _size(X, Y, Z, rows, M, median, hi, scale):
    """N and the mean number of points of a walk (of a sample) for these sizes."""
    dev = _device()
    g = _generator(0, dev)
    centre, brain, semi, at = _anatomy((X, Y, Z), rows)
    shell = _ellipsoid((X, Y, Z), centre, brain, dev) & ~_ellipsoid((X, Y, Z), centre, tuple(max(0.5, a - 3.0) for a in brain), dev)
    N = int(((_ellipsoid((X, Y, Z), at[0], semi, dev) | _ellipsoid((X, Y, Z), at[1], semi, dev)) & ~shell).sum())
    off = _walks((X, Y, Z), rows, 4096, median, hi, scale, g, dev)[1]
    return N, float(off[-1]) / 4096


def _work(case):
    """A point is read once (its two ends only in the seed-to-end mode) and its voxel found, each inserted
    one formed first; offsets are read and C written; a plain call also reads both volumes."""
    N, mean = _size(case["X"], case["Y"], case["Z"], case["rows"], case["M"], case["median"], case["hi"], case.get("scale", 1.0))
    S, up, mode = case["S"], case.get("up", 1), case.get("mode", 0)
    points = 2.0 * S if mode == 3 else S * mean
    nbytes = 12 * points + 8 * (S + 1) + 4 * N * case["M"]
    if case["form"] == "count":
        nbytes += 8 * case["X"] * case["Y"] * case["Z"]
    return nbytes, points * (3 + (3 if case.get("scale", 1.0) != 1.0 else 0) + (3 + 9 * (up - 1) if up > 1 else 0))


def work(case):
    if case["form"] == "parcellate":
        n = case["rows"] * case["M"]
        return {"bytes": 8 * n + 12 * case["rows"], "flops": 2 * n}
    parts = [_work(_shrunk(case, k)) for k in range(case["subjects"])] if "subjects" in case else [_work(case)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ---- the same in plain torch ----

def _distinct_pairs(line, row, lab, S, N, M):
    """C of the hits (line, row) and (line, lab) given as (line, value) pairs of tensors."""
    kr = torch.unique(line[0] * N + row)
    km = torch.unique(line[1] * M + lab)
    lr, lm = kr // N, km // M
    per = torch.bincount(lm, minlength=S)
    first = torch.cumsum(per, 0) - per
    reps = per[lr]
    at = torch.repeat_interleave(torch.arange(kr.numel(), device=kr.device), reps)
    k = torch.arange(at.numel(), device=kr.device) - (torch.cumsum(reps, 0) - reps)[at]
    pair = (kr % N)[at] * M + (km % M)[first[lr[at]] + k]
    return torch.bincount(pair, minlength=N * M)


def _voxels(q, s):
    """Row and label (or -1) of scaled points: the definition's binary32 sum, then an exact floor."""
    t = q + torch.tensor(0.5, dtype=torch.float32, device=q.device)
    Z, Y, X = s["roi"].shape
    ok = (t >= 0).all(1) & (t < torch.tensor([X, Y, Z], dtype=torch.float32, device=q.device)).all(1)
    v = torch.where(ok[:, None], t, torch.zeros_like(t)).to(torch.int64)
    lin = v[:, 0] + X * (v[:, 1] + Y * v[:, 2])
    no = torch.full_like(lin, -1)
    return torch.where(ok, s["roi"].reshape(-1)[lin].to(torch.int64), no), torch.where(ok, s["lab"].reshape(-1)[lin].to(torch.int64), no)


def _exact_count(s):
    S, N, M, off = s["offsets"].numel() - 1, s["N"], s["M"], s["offsets"]
    C = torch.zeros(N * M, dtype=torch.int64, device=off.device)
    step = 1 << 17
    for a in range(0, S, step):
        b = min(S, a + step)
        lo, hi = int(off[a]), int(off[b])
        q = s["points"][lo:hi] * torch.tensor(s["scale"], dtype=torch.float32, device=off.device)
        line = torch.repeat_interleave(torch.arange(b - a, device=off.device), off[a + 1:b + 1] - off[a:b])
        first, last = off[a:b] - lo, off[a + 1:b + 1] - lo - 1
        if s["mode"] == 3:
            r, m = _voxels(q[first], s)[0], _voxels(q[last], s)[1]
            ok = (r >= 0) & (m >= 0)
            C += torch.bincount((r * M + m)[ok], minlength=N * M)
            continue
        lr, rr, lm, mm = [], [], [], []
        for t in range(s["up"]):
            p, of = q, line
            if t:
                f = torch.tensor(np.float32(t / s["up"]), device=q.device)
                same = line[1:] == line[:-1]
                p, of = (q[:-1] + f * (q[1:] - q[:-1]))[same], line[:-1][same]
            r, m = _voxels(p, s)
            lr.append(of[r >= 0])
            rr.append(r[r >= 0])
            if s["mode"] == 0:
                lm.append(of[m >= 0])
                mm.append(m[m >= 0])
        for e in ([last] if s["mode"] == 1 else [first, last] if s["mode"] == 2 else []):
            m = _voxels(q[e], s)[1]
            lm.append(line[e][m >= 0])
            mm.append(m[m >= 0])
        C += _distinct_pairs((torch.cat(lr), torch.cat(lm)), torch.cat(rr), torch.cat(mm), b - a, N, M)
    return C.reshape(N, M)


def exact(case, seed):
    if case["form"] == "parcellate":
        C = _matrix(case, seed).to(torch.int64)
        sums = C.sum(1)
        best, at = C.max(1)
        at = torch.argmax((C == best[:, None]).to(torch.int8), 1)
        frac = C.double() / sums.clamp(min=1).double()[:, None]
        return {"label": torch.where(best > 0, at, torch.full_like(at, -1)), "fractions": frac, "sums": sums}
    if work(case)["bytes"] > 4e9:      # minutes of sorting
        return None
    Cs = [_exact_count(s) for s in _subjects(case, seed)]
    return Cs if case["form"] in ("batched", "served") else Cs[0]
