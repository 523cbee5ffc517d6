"""The offset step's two forms give the same bits.

A launch skins the new pose's surface within the offset step where every
stream in it has its blocks' rims laid out, and in a launch of its own
otherwise, so one mesh in random order (whose rims are too long) switches the
form for the streams served beside it.  Each stream still ends where it ends
alone, over several iterations and frames, for both blends, both solves and
each workgroup size of either form (64, 256 and 512 vertices; 512 only apart
from the skinning)."""
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


def _shuffled(m, rng):
    V = m["rest_xyz"].shape[0]
    order = rng.permutation(V)
    place = np.empty(V, np.int32)
    place[order] = np.arange(V, dtype=np.int32)
    m = dict(m)
    for k in ("rest_xyz", "skin_link", "skin_w"):
        m[k] = np.ascontiguousarray(m[k][order])
    nb = np.asarray(m["neighbors"])[order]
    m["neighbors"] = np.where(nb >= 0, place[nb], -1).astype(np.int32)
    m["faces"] = place[m["faces"]]
    return m


def _stream(body, model, seed):
    """(model, camera, theta0, offsets, frames)"""
    rng = np.random.default_rng(seed)
    P, V = len(model["joint_parent"]), model["rest_xyz"].shape[0]
    th = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    frames = []
    for f in range(2):
        t = th + np.where(body.angular, 0.01 * f, 0.001 * f)
        frames.append(synth.render_frame(model, body.camera, synth.pose_surface(model, t), rng, 0.2, 0.002))
    return (model, body.camera, th + np.where(body.angular, 0.02, 0.002),
            rng.normal(0, 0.0005, (V, 3)).astype(np.float32), frames)


def _alone(T, prm, s):
    model, cam, th0, phi0, frames = s
    trk = T.Tracker(model, cam, prm, th0, phi0)
    try:
        for d in frames:
            assert trk.frame(d) == 0, T.track_last_error()
        return trk.state(want_verts=False)[:2]
    finally:
        trk.close()


def _together(T, prm, streams):
    sv = T.track_server_create(prm, 1 << 36, 8)
    try:
        ids = []
        for model, cam, th0, phi0, frames in streams:
            ids.append(T.track_server_open(sv, model, cam, th0, phi0))
            for d in frames:
                T.track_server_submit(sv, ids[-1], d)
        left = sum(len(s[4]) for s in streams)
        for _ in range(100):
            T.track_server_step(sv)
            for c in T.track_server_poll(sv):
                assert c["status"] == 0, c
                left -= 1
            if left == 0:
                break
        assert left == 0
        return [T.track_server_state(sv, i, len(s[0]["joint_parent"]), s[0]["rest_xyz"].shape[0])
                for i, s in zip(ids, streams)]
    finally:
        T.track_server_destroy(sv)


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("blend", [0, 1])
@pytest.mark.parametrize("ring,rings", [(9, 7), (37, 54), (129, 127), (362, 361)])
def test_served_beside_a_mesh_of_long_rims(T, ring, rings, blend, fp64):
    body, other = synth.make_arm(ring, rings), synth.make_arm(37, 54)
    rng = np.random.default_rng(ring)
    mine = dict(body.model, blend=blend)
    long_rims = dict(_shuffled(other.model, rng), blend=blend)
    print(f"[shape forms] {mine['rest_xyz'].shape[0]} vertices blend={blend} fp64={fp64}", flush=True)
    prm = dict(synth.default_params(len(mine["joint_parent"]), 4, 0.05, lambda_t=0.5, lambda_k=0.1),
               shape_solve_fp64=fp64, active=None)
    streams = [_stream(body, mine, 1), _stream(other, long_rims, 2)]
    got = _together(T, prm, streams)
    for s, (th, phi) in zip(streams, got):
        th_a, phi_a = _alone(T, prm, s)
        assert np.abs(phi - s[3]).max() > 0
        np.testing.assert_array_equal(th, th_a)
        np.testing.assert_array_equal(phi, phi_a)
