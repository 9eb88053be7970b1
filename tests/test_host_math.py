"""Host tests of arithmetic that the kernels share with the host (csrc/internal.h), built here for the CPU
(tests/native/host_math.hip): which voxels of a row a lane of the compact build reads and owns;
that one 32-bit code holds every row and label that the argument checks let in; which range of the points
a streamline belongs to, of which the table of ranges needs that it never decreases; that the ranges which
wavefronts find for themselves cover every streamline once; that a plan's preparation gives every subject
workgroups in proportion to its work."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_math") / "libhost_math.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-fPIC", "-shared",
                           "-Wall", "-Werror", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2302_09247_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "host_math.hip"), "-o", out])
    return ctypes.CDLL(out)


@pytest.mark.parametrize("wide", [0, 1])
def test_build_lanes_own_every_voxel_of_a_row_once(lib, wide):
    out = (ctypes.c_int32 * 3)()
    for X in list(range(4 if wide else 1, 140)) + ([] if not wide else [255, 256, 257, 311]):
        if not wide and X >= 4:
            continue   # rows of at least 4 voxels take the wide loads
        owners = np.zeros(X, np.int64)
        for x in range(0, (X + 127) // 128 * 128, 4):   # a workgroup's lanes cover 128 voxels along x
            lib.row_lane(wide, x, X, out)
            xs, d, mine = out[0], out[1], out[2]
            assert 0 <= d <= 3, (X, x, d)               # the lane's bits are shifted by d in every lane
            assert 0 <= xs and (not wide or xs + 4 <= X), (X, x, xs)   # (narrow loads are clamped one by one)
            for i in range(4):
                if (mine >> i) & 1:
                    assert xs + i == x + i - d and i >= d
                    owners[xs + i] += 1
        assert (owners == 1).all(), X


def _shapes():
    for rb in range(1, 32):
        for n in (1 << (rb - 1), (1 << rb) - 1):
            most = ((1 << 31) - 1) // n                     # N * M < 2^31
            for m in {1, 2, most // 2, most - 1, most, 1 << (most.bit_length() - 1)}:
                if 1 <= m <= most:
                    yield n, m


def test_a_code_of_32_bits_holds_every_row_and_label(lib):
    out = (ctypes.c_int64 * 4)()
    dims = (ctypes.c_int32 * 3)(30, 20, 10)
    for N, M in _shapes():
        assert lib.layout(dims, N, M, out) == 1, (N, M)
        rbits, rmask = out[0], out[1]
        assert out[2] == out[3] + 4 * 30 * 20 * 10          # 4 bytes a code
        none = 0xFFFFFFFF
        # "none" in either field is no row and no label, and the largest of both come back as they went in
        assert none & rmask >= N and none >> rbits >= M
        code = (N - 1) | ((M - 1) << rbits)
        assert code < 1 << 32 and code & rmask == N - 1 and code >> rbits == M - 1, (N, M)


def _ranges(lib, P, nparts, equal, p):
    p = np.ascontiguousarray(p, np.int64)
    out = np.empty(p.size, np.int32)
    lib.range_of(ctypes.c_int64(P), ctypes.c_int64(nparts), equal, p.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(p.size),
                 out.ctypes.data_as(ctypes.c_void_p))
    return out.astype(np.int64)


POINTS = [0, 1, 2, 5, 999, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 25) - 1, 1 << 25, 3 * (1 << 24) + 7, 112_532_461,
          1_097_713_418, (1 << 32) - 1, 1 << 32, (1 << 32) + 1, (1 << 36) + 12345, (1 << 40) - 1, 1 << 40]


@pytest.mark.parametrize("equal", [0, 1])
@pytest.mark.parametrize("P", POINTS)
def test_ranges_never_decrease(lib, P, equal):
    rng = np.random.default_rng(P % 1000 + equal)
    p = rng.integers(0, P + 1, 200_000) if P > 200_000 else np.arange(P + 1)
    step = max(1, P >> 24)
    edges = np.concatenate([[0, P], (rng.integers(0, P + 1, 2000) // step * step)[:, None].repeat(3, 1).ravel() + np.tile([-1, 0, 1], 2000)])
    p = np.sort(np.concatenate([p, np.clip(edges, 0, P), [-5, P + 5]]))
    for nparts in (1, 2, 3, 7, 64, 1000, 6144, 28_672, 49_152, 50_001):
        r = _ranges(lib, P, nparts, equal, p)
        assert (np.diff(r) >= 0).all(), nparts
        assert r[0] == 0 and r.max() < nparts
        if P > 1 << 20:   # range i holds about the share of the points it should (24-bit positions: to 1 in 300)
            i = np.arange(nparts + 1) / nparts
            want = P * (i if equal else 1.5 * i - 0.5 * i * i)
            got = p[np.searchsorted(r, np.arange(nparts))]
            spread = P / 200_000 * 30 + P / nparts
            assert np.abs(got - want[:-1]).max() < spread
            assert r[-1] == nparts - 1


@pytest.mark.parametrize("seed", range(6))
def test_one_pass_writes_every_range_once(lib, seed):
    # the table's rule: streamline s writes the ranges in (range(s - 1), range(s)], the end of the last
    # streamline those that are left, nparts included; a plan's items: the last streamline takes the rest
    rng = np.random.default_rng(seed)
    S = int(rng.choice([1, 2, 63, 64, 65, 5000, 40_000]))
    lens = rng.integers(0, 200, S)
    lens[rng.random(S) < 0.3] = 0
    lens[: S // 7] = 0
    lens[S - S // 7:] = 0
    if seed % 2:
        lens[S // 2] = 1 + 1000 * S
        lens[S // 3: S // 3 + 40] *= 300
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64) * (1 if seed < 4 else 70_001)
    for nparts in (1, 2, 5, 64, 6144, 28_672):
        r = _ranges(lib, int(off[-1]), nparts, 0, off[:-1])
        hi = np.append(r, nparts)
        lo = np.append(-1, r) + 1
        first = np.full(nparts + 1, -1)
        writes = np.zeros(nparts + 1, np.int64)
        for s in range(S + 1):
            first[lo[s]:hi[s] + 1] = s
            writes[lo[s]:hi[s] + 1] += 1
        assert (writes == 1).all() and first[0] == 0 and first[-1] == S and (np.diff(first) >= 0).all()
        # every streamline is in the range it belongs to
        for i in rng.integers(0, nparts, 50):
            assert (r[first[i]:first[i + 1]] == i).all()
        e = _ranges(lib, int(off[-1]), nparts, 1, off[:-1])
        hi = e.copy()
        hi[-1] = nparts - 1
        lo = np.append(-1, e[:-1]) + 1
        writes = np.zeros(nparts, np.int64)
        for s in range(S):
            writes[lo[s]:hi[s] + 1] += 1
        assert (writes == 1).all()


@pytest.mark.parametrize("width", [256, 1024])
@pytest.mark.parametrize("seed", range(4))
def test_count_search_of_either_workgroup_size(width, seed):
    # the overflow queue's search for a point's streamline runs in workgroups of 256 threads, and of 1024
    # beside the sorting of the pair buffer: `width` evenly spaced offsets a round
    rng = np.random.default_rng(100 * width + seed)
    S = int(rng.choice([1, 2, width - 1, width, width + 1, 70_000, 3_000_000]))
    lens = rng.integers(0, 400, S)
    lens[rng.random(S) < 0.2] = 0
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    if off[-1] == 0:
        return
    for p in rng.integers(0, off[-1], 100):
        lo, hi = 0, S
        while hi - lo > 1:
            step = (hi - lo + width - 1) // width
            at = lo + np.arange(1, width, dtype=np.int64) * step
            lo += int((off[at[at < hi]] <= p).sum()) * step
            hi = min(hi, lo + step)
        assert lo == int(np.searchsorted(off, p, side="right")) - 1 and off[lo] <= p < off[lo + 1]


def _own_ranges(off, nparts):
    """numpy model of the ranges that wavefronts find for themselves (one per wavefront, no table)."""
    S = off.size - 1
    P = max(int(off[-1]), 0)
    ln = int(np.float64(P) * (1.0 / np.float64(S))) + 1
    inv = 1.0 / np.float64(nparts)

    def target(w):
        return int(np.float64(P + ln * S) * (np.float64(w) * inv))

    def first_at(w):
        lo, hi, t, rounds = 0, S, target(w), 0
        while lo < hi:
            step = (hi - lo + 63) // 64
            at = lo + np.arange(64, dtype=np.int64) * step
            at = at[at < hi]
            n = int((off[at] + ln * at < t).sum())
            hi = min(hi, lo + n * step) if n else lo
            lo = lo + (n - 1) * step + 1 if n else lo
            rounds += 1
            assert 0 <= lo <= hi <= S and rounds <= 6
        return lo

    out = []
    for w in range(nparts):
        s0 = 0 if w == 0 else first_at(w)
        s1 = S
        if w + 1 < nparts:
            at = np.arange(s0, s0 + 64)
            at = at[at < S]
            n = int((off[at] + ln * at < target(w + 1)).sum())
            s1 = s0 + n if n < 64 else max(s0, first_at(w + 1))
        out.append((s0, s1))
    return out, ln


@pytest.mark.parametrize("order", ["drawn", "sorted", "falling", "long in a row", "empty runs", "giant"])
@pytest.mark.parametrize("S,nparts", [(3, 1), (200, 64), (2049, 1024), (5000, 1024), (32_768, 1024), (20_000, 8192)])
def test_own_ranges_cover_every_streamline_once(order, S, nparts):
    rng = np.random.default_rng(S + len(order))
    lens = np.clip(np.round(150 * np.exp(0.5 * rng.standard_normal(S))), 20, 600).astype(np.int64)
    if order == "sorted":
        lens.sort()
    if order == "falling":
        lens = np.sort(lens)[::-1].copy()
    if order == "long in a row":
        lens[: S // 20] *= 10
    if order == "empty runs":
        lens[: S // 4] = 0
        lens[S - S // 4:] = 0
        lens[rng.random(S) < 0.3] = 0
    if order == "giant":
        lens[S // 2] = 1 << 40
    off = np.concatenate([[0], np.cumsum(lens)])
    ranges, ln = _own_ranges(off, nparts)
    assert ranges[0][0] == 0 and ranges[-1][1] == S
    assert all(a[1] == b[0] for a, b in zip(ranges, ranges[1:]))
    # at most twice the mean of the streamlines, and of the points but for the last one's length
    per = np.array([b - a for a, b in ranges])
    assert per.max() <= 2 * S / nparts + 2
    begun = np.array([off[b - 1] - off[a] if b > a else 0 for a, b in ranges])
    assert begun.max() <= 2 * (off[-1] + S) / nparts + 2


@pytest.mark.parametrize("seed", range(4))
def test_own_ranges_of_decreasing_offsets_stay_in_bounds(seed):
    # malformed offsets give wrong counts, but every range lies in [0, S] and the search ends
    rng = np.random.default_rng(seed)
    S = 4000
    off = rng.integers(-1000 if seed % 2 else 0, 300_000, S + 1)
    for s0, s1 in _own_ranges(off, 512)[0]:
        assert 0 <= s0 <= s1 <= S


def _grid(lib, work, nzero=5200, cus=256):
    w = np.asarray(work, np.int64)
    base = np.zeros(w.size + 1, np.int64)
    vp = ctypes.c_void_p
    t = lib.prepare_grid(w.ctypes.data_as(vp), ctypes.c_int32(w.size), ctypes.c_int64(nzero), ctypes.c_int(cus), base.ctypes.data_as(vp))
    assert t >= 0
    return (np.diff(base) if t else np.full(w.size, base[0])), base, bool(t)


@pytest.mark.parametrize("small", [0, 1, 100, 3000])
@pytest.mark.parametrize("n", [1, 2, 16, 64, 256, 1000, 5000])
@pytest.mark.parametrize("big", [100, 20_000, 3_000_000, 20_000_000])
def test_preparation_workgroups_follow_the_work(lib, small, n, big):
    for at in {0, n // 2, n - 1}:
        work = np.full(n, small, np.int64)
        work[at] = big
        blocks, base, table = _grid(lib, work)
        assert ((blocks >= 1) | (work == 0)).all()
        assert blocks.sum() <= 4096 + n or not table
        # no subject needs more than about twice the steps of an even split over the whole launch
        steps = np.ceil(work / np.maximum(blocks, 1) / 256)
        even = np.ceil(work.sum() / (4096 * 256))
        assert steps.max() <= 2 * even + 2, (steps.max(), even, table)
        if table:   # every workgroup finds its subject (64 bases a round)
            for b in np.unique(np.concatenate([[0, base[n] - 1], base[:-1][blocks > 0], base[1:][blocks > 0] - 1])):
                lo, hi = 0, n
                while hi - lo > 1:
                    step = (hi - lo + 63) // 64
                    idx = lo + np.arange(64) * step
                    lo += (int((base[idx[idx < hi]] <= b).sum()) - 1) * step
                    hi = min(hi, lo + step)
                assert base[lo] <= b < base[lo + 1], (b, lo)


def test_balanced_plans_keep_equal_shares(lib):
    rng = np.random.default_rng(5)
    for n in (1, 12, 24, 100):
        assert not _grid(lib, rng.integers(100_000, 300_000, n))[2]
