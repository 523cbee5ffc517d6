"""A state cannot be read while the caller captures the stream: the call is
refused, puts nothing into the graph, and does not take the surface for
skinned, so the next read gives the true one."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_reading_under_capture_is_refused():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track as T

    body = synth.make_arm(16, 8)
    m, cam, P, V = body.model, body.camera, len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    rng = np.random.default_rng(3)
    th = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    depth = synth.render_frame(m, cam, synth.pose_surface(m, th), rng, 0.0, 0.0)
    prm = synth.default_params(P, 2, 0.05)
    stream = torch.cuda.Stream()
    mine, other = T.Tracker(m, cam, prm, 0.9 * th, stream=stream.cuda_stream), T.Tracker(m, cam, prm, 0.9 * th)
    hip = ctypes.CDLL(T.LIB_PATH)   # (its own HIP runtime, whatever the path)
    try:
        for trk in (mine, other):
            assert trk.frame(depth) == 0, T.track_last_error()
        want = other.state()
        print("[state] read under capture", flush=True)
        graph, n = ctypes.c_void_p(), ctypes.c_size_t(1)
        s = ctypes.c_void_p(stream.cuda_stream)
        assert hip.hipStreamBeginCapture(s, 1) == 0   # thread-local
        try:
            with pytest.raises(T.TrackError) as e:
                mine.state()
        finally:
            ended = hip.hipStreamEndCapture(s, ctypes.byref(graph))
        assert e.value.code == T.TRACK_E_DEVICE
        assert ended == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == 0
        hip.hipGraphDestroy(graph)
        got = mine.state()
        for a, b in zip(got[:3], want[:3]):
            np.testing.assert_array_equal(a, b)
    finally:
        mine.close()
        other.close()
