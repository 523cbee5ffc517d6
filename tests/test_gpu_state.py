"""The state as it reaches the caller against the buffers themselves, for
vertex counts that leave every remainder of the 16-byte pieces it travels in,
before and after a frame."""
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


@pytest.mark.parametrize("ring,rings", [(9, 7), (16, 8), (9, 9), (8, 9), (37, 54), (129, 127)])   # 65, 130, 83, 74, ...
def test_state_is_what_the_buffers_hold(T, ring, rings):
    body = synth.make_arm(ring, rings)
    m, cam, P, V = body.model, body.camera, len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    print(f"[state] {V} vertices", flush=True)
    rng = np.random.default_rng(V)
    th0 = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    depth = synth.render_frame(m, cam, synth.pose_surface(m, th0), rng, 0.0, 0.0)
    phi0 = rng.normal(0, 0.001, (V, 3)).astype(np.float32)
    trk = T.Tracker(m, cam, synth.default_params(P, 2, 0.05), 0.9 * th0)
    try:
        trk.reset(0.9 * th0, phi0)
        th, phi, v, _ = trk.state()
        np.testing.assert_array_equal(th, 0.9 * th0)
        np.testing.assert_array_equal(phi, phi0)
        for frame in range(2):
            assert trk.frame(depth) == 0, T.track_last_error()
            th, phi, none, _ = trk.state(want_verts=False)
            assert none is None
            th2, phi2, v, _ = trk.state()
            np.testing.assert_array_equal(th, th2)
            np.testing.assert_array_equal(phi, phi2)
            np.testing.assert_array_equal(th, T.track_dbg_get(trk.ctx, T.TRACK_BUF_THETA, (P,), np.float64))
            np.testing.assert_array_equal(phi, T.track_dbg_get(trk.ctx, T.TRACK_BUF_PHI, (V, 3), np.float32))
            np.testing.assert_array_equal(v, T.track_dbg_get(trk.ctx, T.TRACK_BUF_VERTS, (V, 3), np.float32))
    finally:
        trk.close()


def test_threads_read_states_of_one_server(T):
    """States of a server's streams read by several threads at once are each
    the stream's own."""
    from concurrent.futures import ThreadPoolExecutor

    body = synth.make_arm(37, 54)
    m, cam, P, V = body.model, body.camera, len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    rng = np.random.default_rng(1)
    sv = T.track_server_create(dict(synth.default_params(P, 1, 0.05), active=None), 1 << 34, 8)
    try:
        ths = [rng.uniform(-0.1, 0.1, P) for _ in range(6)]
        phis = [rng.normal(0, 0.001, (V, 3)).astype(np.float32) for _ in range(6)]
        ids = [T.track_server_open(sv, m, cam, th, phi) for th, phi in zip(ths, phis)]
        print("[state] six streams, four threads", flush=True)
        with ThreadPoolExecutor(4) as pool:
            got = list(pool.map(lambda k: (k, T.track_server_state(sv, ids[k], P, V)), [k % 6 for k in range(60)]))
        for k, (th, phi) in got:
            np.testing.assert_array_equal(th, ths[k])
            np.testing.assert_array_equal(phi, phis[k])
    finally:
        T.track_server_destroy(sv)
