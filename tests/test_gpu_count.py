"""The bucket index as the skinning and the offset step count it, for each
workgroup size they are launched with (64, 256 and 512 vertices, chosen by the
vertex count) and vertex counts that leave a remainder: the association of
the surface each of them counted is bit-exact against the oracle's on that
surface."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


# (vertices around, along): 65, 16385 and 130684 vertices
@pytest.mark.parametrize("ring,rings", [(9, 7), (129, 127), (362, 361)])
def test_counted_surfaces_associate_bit_exact(T, ring, rings):
    body = synth.make_arm(ring, rings)
    cam, V, P = body.camera, body.model["rest_xyz"].shape[0], len(body.model["joint_parent"])
    print(f"[count] {V} vertices", flush=True)
    rng = np.random.default_rng(V)
    th = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    depth = synth.render_frame(body.model, cam, synth.pose_surface(body.model, th), rng, 0.2, 0.002)
    prm = synth.default_params(P, 2, 0.05)
    for shape in ([0, 0], [1, 0]):   # the second association reads the frame start's count, or the offset step's
        p = dict(prm, do_pose=np.zeros(2, np.uint8), do_shape=np.array(shape, np.uint8))
        trk = T.Tracker(body.model, cam, p, th)
        try:
            for _ in range(2):   # the second frame in the layout the first left
                assert trk.frame(depth) == 0, T.track_last_error()
                got = T.track_dbg_get(trk.ctx, T.TRACK_BUF_ASSOC, (cam["height"] * cam["width"],), np.int32)
                verts = trk.state()[2]
                want = oracle.associate(cam, prm["tau"], verts, depth=depth)
                assert (want >= 0).sum() > 100
                np.testing.assert_array_equal(got, want)
        finally:
            trk.close()
