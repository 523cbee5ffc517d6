"""Reading a state neither reports nor takes an error that another of the
thread's HIP calls left."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_an_earlier_error_stays_the_callers():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track as T

    body = synth.make_arm(9, 7)
    m, cam, P, V = body.model, body.camera, len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    prm = synth.default_params(P, 1, 0.05)
    th = np.linspace(-0.1, 0.1, P)
    trk = T.Tracker(m, cam, prm, th)
    sv = T.track_server_create(dict(prm, active=None), 1 << 32, 2)
    hip = ctypes.CDLL(T.LIB_PATH)   # (its own HIP runtime, whatever the path)
    try:
        sid = T.track_server_open(sv, m, cam, th)
        hip.hipGetLastError()
        print("[state] a device that does not exist", flush=True)
        left = hip.hipSetDevice(1 << 20)
        assert left != 0 and hip.hipPeekAtLastError() == left
        np.testing.assert_array_equal(trk.state()[0], th)
        np.testing.assert_array_equal(T.track_server_state(sv, sid, P, V)[0], th)
        assert hip.hipGetLastError() == left
        assert hip.hipGetLastError() == 0
    finally:
        hip.hipGetLastError()
        T.track_server_destroy(sv)
        trk.close()
