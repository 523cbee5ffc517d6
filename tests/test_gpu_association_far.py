"""The association's depth filter at long range, where a cutoff is a few
hundred to a few thousand units in the last place of the depths: vertices
straight behind (or before) their pixels at the largest depth difference that
is still below the cutoff, as float32 subtracts it.  Every cell of vertices
lies at one depth, so that a filter by the cells' depth ranges decides about
exactly that difference.  Bit-exact against the oracle's exhaustive search."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


# depth, steps of a float32 there up to the cutoff
@pytest.mark.parametrize("z,steps", [(1.5, 40000), (12.0, 5000), (20.0, 1500), (33.0, 1000), (50.0, 2000), (100.0, 450)])
def test_just_below_the_cutoff(T, tiny, z, steps):
    W, H, f = 62, 45, 70.0
    print(f"[far] {z} m, {steps} steps", flush=True)
    ulp = np.spacing(np.float32(z))
    tau = np.nextafter(np.float32(steps * ulp), np.float32(np.inf))
    cam = dict(width=W, height=H, fx=f, fy=f, cx=(W - 1) / 2.0, cy=(H - 1) / 2.0)
    V = tiny.body.model["rest_xyz"].shape[0]
    rng = np.random.default_rng(steps)
    pix = rng.choice(W * H, V, replace=False)
    u, v = (pix % W).astype(np.float32), (pix // W).astype(np.float32)
    d = np.float32(z)
    far = u >= W // 2   # a vertex behind its pixel on the right, before it on the left
    verts = np.stack([((u - np.float32(cam["cx"])) * d) / np.float32(f), ((v - np.float32(cam["cy"])) * d) / np.float32(f),
                      np.where(far, d + np.float32(steps) * ulp, d - np.float32(steps) * ulp)], 1).astype(np.float32)
    depth = np.full((H, W), d, np.float32)
    depth[rng.random((H, W)) < 0.1] = 0.0
    want = oracle.associate(cam, float(tau), verts, depth=depth, brute=True)
    assert (want >= 0).sum() > V // 2
    trk = T.Tracker(tiny.body.model, cam, dict(tiny.params, tau=float(tau)), tiny.theta0)
    try:
        T.track_dbg_set(trk.ctx, T.TRACK_BUF_VERTS, verts)
        T.track_dbg_set(trk.ctx, T.TRACK_BUF_DEPTH, depth)
        assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_ASSOCIATE) == 0
        got = T.track_dbg_get(trk.ctx, T.TRACK_BUF_ASSOC, (W * H,), np.int32)
    finally:
        trk.close()
    np.testing.assert_array_equal(got, want)
