"""The offset step that skins the new pose's surface itself, over blocks of 64
vertices and their rims: a block and one vertex, a rim short of a full round,
vertices of more than eight faces (the tube's poles), both workgroup sizes
that take this form, and a mesh in random order, whose rims are too long and
which therefore skins in a launch of its own."""
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


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("ring,rings,shuffle", [(9, 7, False), (37, 54, False), (37, 54, True), (129, 127, False)])
def test_step_after_a_pose_step(T, ring, rings, shuffle, fp64):
    """One iteration (pose, then offsets) against the oracle's offset step at
    the pose and the matches that it left.  The float32 surface is within 16
    ulp of the oracle's, so a normal is off by 16 ulp (1 m) / the shortest
    edge (1.8 mm), 5e-4 at most, and a residual by that share of the vertex'
    mean offset and by 32 ulp (surface, mean offset, products); both enter the
    step divided by the regulariser's weight, the former twice (the step's
    direction is the normal's)."""
    body = synth.make_arm(ring, rings)
    m, cam, P = body.model, body.camera, len(body.model["joint_parent"])
    rng = np.random.default_rng(ring + rings)
    if shuffle:
        m = _shuffled(m, rng)
    V = m["rest_xyz"].shape[0]
    print(f"[shape rims] {V} vertices shuffle={shuffle} fp64={fp64}", flush=True)
    th = np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P))
    depth = synth.render_frame(m, cam, synth.pose_surface(m, th), rng, 0.1, 0.0)
    prm = dict(synth.default_params(P, 1, 0.05, lambda_t=0.5), shape_solve_fp64=fp64)
    phi0 = rng.normal(0, 0.0005, (V, 3)).astype(np.float32)
    th0 = th + np.where(body.angular, 0.01, 0.001)
    trk = T.Tracker(m, cam, prm, th0, phi0)
    try:
        assert trk.frame(depth) == 0, T.track_last_error()
        th1, phi1 = trk.state(want_verts=False)[:2]
        match = T.track_dbg_get(trk.ctx, T.TRACK_BUF_ASSOC, (cam["height"] * cam["width"],), np.int32)
    finally:
        trk.close()
    assert (match >= 0).sum() > 100
    v0 = oracle.skin(m, th0, phi0.astype(np.float64))[0]
    cnt, delta = oracle.average(cam, match, v0, depth=depth)
    v1, n1 = oracle.skin(m, th1, phi0.astype(np.float64))
    d1 = np.where(cnt[:, None] > 0, delta + (v0 - v1), delta)
    want = oracle.shape_step(m, th1, phi0.astype(np.float64), phi0.astype(np.float64), n1, d1, cnt, prm["lambda_phi"],
                             prm["lambda_nbr"], prm["lambda_t"], prm["lambda_w"])
    alpha = prm["lambda_phi"] + prm["lambda_t"] + prm["lambda_nbr"] * (np.asarray(m["neighbors"]) >= 0).sum(axis=1)
    off = np.where(cnt > 0, np.linalg.norm(d1, axis=1), 0.0)
    tol = (1e-3 * off + 32 * float(np.spacing(np.float32(1.0)))) / alpha + 1e-3 * np.abs(want - phi0).max(axis=1)
    err = np.abs(phi1 - want).max(axis=1)
    print(f"  error over bound at most {np.max(err / tol):.2f}", flush=True)
    assert (err <= tol).all()
