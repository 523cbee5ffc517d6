"""What a resident stream takes of a server's budget: no more than before the
offset step's and the normal equations' per-stream tables came (the sizes
measured then), so that a budget holds the streams it held.  And streams that
had to wait, whose tables are made a second time, end where they end alone."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


CAM = dict(width=640, height=480, fx=525.0, fy=525.0, cx=319.5, cy=239.5)


@pytest.mark.parametrize("verts,before", [(2000, 1353728), (3000, 11147520), (50000, 37089024), (200000, 92983040)])
def test_bytes_of_a_stream(T, verts, before):
    body = synth.make_arm() if verts == 2000 else synth.make_body(verts, CAM, 2.6)
    cam = body.camera if verts == 2000 else CAM
    P = len(body.model["joint_parent"])
    sv = T.track_server_create(dict(synth.default_params(P, 2, 0.05), active=None), 1 << 34, 2)
    try:
        T.track_server_open(sv, body.model, cam, np.zeros(P))
        used = T.track_server_info(sv)["bytes_used"]
    finally:
        T.track_server_destroy(sv)
    print(f"[memory] {verts} vertices: {used} bytes, {before} before", flush=True)
    assert used <= before


def test_streams_that_waited(T):
    body = synth.make_arm(37, 54)
    P, V = len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    prm = synth.default_params(P, 3, 0.05, lambda_k=0.1)
    rng = np.random.default_rng(5)
    th = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    depth = synth.render_frame(body.model, body.camera, synth.pose_surface(body.model, th), rng, 0.2, 0.002)
    th0 = [th + np.where(body.angular, 0.01 * k, 0.001 * k) for k in range(1, 4)]
    sv = T.track_server_create(dict(prm, active=None), 1 << 34, 1)   # one resident stream
    try:
        ids = [T.track_server_open(sv, body.model, body.camera, t) for t in th0]
        assert T.track_server_info(sv)["waiting"] == 2
        for i in ids:
            T.track_server_submit(sv, i, depth)
        got = []
        for i in ids:
            for _ in range(prm["n_iters"]):
                T.track_server_step(sv)
            assert [c["status"] for c in T.track_server_poll(sv)] == [0]
            got.append(T.track_server_state(sv, i, P, V))
            T.track_server_close(sv, i)
    finally:
        T.track_server_destroy(sv)
    for t, (a, b) in zip(th0, got):
        trk = T.Tracker(body.model, body.camera, prm, t)
        try:
            assert trk.frame(depth) == 0, T.track_last_error()
            want = trk.state(want_verts=False)
        finally:
            trk.close()
        np.testing.assert_array_equal(a, want[0])
        np.testing.assert_array_equal(b, want[1])
