"""Host tests of arithmetic that the kernels share with the host (csrc/internal.h), built here for the CPU
(tests/native/host_math.hip): which voxels of a row a lane of the compact build reads and owns."""
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
