"""Host tests of arithmetic that the kernels share with the host (csrc/internal.h), built here for the CPU
(tests/native/host_math.hip): which voxels of a row a lane of the compact build reads and owns;
that one 32-bit code holds every row and label that the argument checks let in."""
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
