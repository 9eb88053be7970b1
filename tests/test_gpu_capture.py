"""GPU tests of counts against a resident volume under stream capture and while its build is pending.

A captured count must give the eager result on every replay, whether or not an eager call has used the
volume before; and a call made while the build is still running must treat an error that its caller
left in the runtime as one made afterwards does.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2302_09247_amd import synth

pytestmark = pytest.mark.gpu


def _raw_count(fc, vol, w, C, stream, noalloc=False):
    lib = fc.load()
    f = lib.fastcod_volume_count_noalloc if noalloc else lib.fastcod_volume_count
    vp = ctypes.c_void_p
    f.argtypes = [vp, vp, vp, ctypes.c_int64, vp, ctypes.POINTER(fc.Opts), vp]
    f.restype = ctypes.c_int
    o = lib.fastcod_default_opts()
    return f(vol.handle, w.points.data_ptr(), w.offsets.data_ptr(), int(w.offsets.shape[0]) - 1, C.data_ptr(),
             ctypes.byref(o), stream.cuda_stream)


@pytest.mark.parametrize("noalloc", [True, False])
@pytest.mark.parametrize("used_before", [False, True])
def test_captured_count_replays(fc, noalloc, used_before):
    w = synth.make_tiny64(seed=31, S=3000, device="cuda")
    exp = oracle.count(w.points, w.offsets, w.roi, w.lab, w.N, w.M)
    vol = fc.Volume(w.roi, w.lab, w.N, w.M)
    C = torch.zeros((w.N, w.M), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    other = fc.Volume(w.roi, w.lab, w.N, w.M)
    if not noalloc:   # the stream's workspace, made by a count against another volume
        assert _raw_count(fc, other, w, C, s) == fc.OK
    if used_before:
        assert _raw_count(fc, vol, w, C, s, noalloc) == fc.OK
    torch.cuda.synchronize()
    print(f"capture noalloc={noalloc} used_before={used_before}", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        rc = _raw_count(fc, vol, w, C, s, noalloc)
    assert rc == fc.OK, fc.load().fastcod_last_error()
    for rep in range(3):
        C.fill_(77 + rep)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(C.cpu().numpy(), exp, err_msg=f"replay {rep}")
        # eager work between the replays, through the same scratch
        D = torch.empty_like(C)
        assert _raw_count(fc, other, w, D, s, noalloc) == fc.OK
        torch.cuda.synchronize()
        np.testing.assert_array_equal(D.cpu().numpy(), exp)
    del g
    vol.close()
    other.close()


def test_a_callers_error_counts_the_same_before_and_after_the_build(fc):
    hip = ctypes.CDLL("libamdhip64.so")
    w = synth.make_tiny64(seed=32, S=2000, device="cuda")
    exp = oracle.count(w.points, w.offsets, w.roi, w.lab, w.N, w.M)
    C = torch.zeros((w.N, w.M), dtype=torch.int32, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    warm = fc.Volume(w.roi, w.lab, w.N, w.M)   # s2's workspace
    assert _raw_count(fc, warm, w, C, s2) == fc.OK
    torch.cuda.synchronize()
    hip.hipGetLastError()
    with torch.cuda.stream(s1):
        torch.cuda._sleep(200_000_000)         # about 0.1 s of work before the build
        vol = fc.Volume(w.roi, w.lab, w.N, w.M)
    hip.hipSetDevice(1_000_000)                # refused: leaves an error
    pending = _raw_count(fc, vol, w, C, s2)
    assert not s1.query()                      # the build was indeed pending
    torch.cuda.synchronize()
    hip.hipGetLastError()
    assert _raw_count(fc, vol, w, C, s2) == fc.OK
    torch.cuda.synchronize()
    np.testing.assert_array_equal(C.cpu().numpy(), exp)
    hip.hipSetDevice(1_000_000)
    built = _raw_count(fc, vol, w, C, s2)
    hip.hipGetLastError()
    print(f"status with a caller's error: build pending {pending}, built {built}", flush=True)
    assert pending == built
    assert _raw_count(fc, vol, w, C, s2) == fc.OK
    torch.cuda.synchronize()
    np.testing.assert_array_equal(C.cpu().numpy(), exp)
    vol.close()
    warm.close()
