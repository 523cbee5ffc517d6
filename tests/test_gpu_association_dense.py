"""Cells of many vertices, which a search compares on their own before it
decides about the eight around them and the rest of its window: cells that hold
one vertex less than that takes, just as many, one more and several passes of
candidates, next to empty and to sparse ones, with pixels that match in their
own cell, in a neighbour, further out, and nowhere.  Bit-exact against the
oracle's exhaustive search, with every vertex in the overflow list (the first
association) and in the cells' regions (the next ones)."""
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


# vertices of a full cell, every how many cells one is full, focal length (the window's width), spread in depth
@pytest.mark.parametrize("full,every,f,spread", [(255, 1, 90.0, 0.02), (256, 1, 90.0, 0.02), (257, 1, 90.0, 0.02),
                                                 (256, 2, 90.0, 0.2), (650, 1, 90.0, 0.05), (330, 2, 400.0, 0.1),
                                                 (1998, 1, 200.0, 0.05)])
def test_dense_cells(T, tiny, full, every, f, spread):
    W, H, tau, z0 = 61, 46, 0.1, 2.0
    print(f"[dense] {full} a cell, every {every}, f = {f}", flush=True)
    cam = dict(width=W, height=H, fx=f, fy=f * 1.01, cx=(W - 1) / 2.0, cy=(H - 1) / 2.0)
    V = tiny.body.model["rest_xyz"].shape[0]
    rng = np.random.default_rng(full + every)
    left, u, v = V, [], []
    for k in range(100):   # cells from the image's middle on, row by row
        if left == 0:
            break
        n = min(left, full if k % every == 0 else 3)
        cx, cy = 6 + k % 4, 4 + k // 4
        u.append(rng.uniform(4 * cx - 0.45, 4 * cx + 3.45, n))
        v.append(rng.uniform(4 * cy - 0.45, 4 * cy + 3.45, n))
        left -= n
    u, v = np.concatenate(u), np.concatenate(v)
    z = rng.uniform(z0, z0 + spread, V)
    verts = np.stack([(u - cam["cx"]) * z / cam["fx"], (v - cam["cy"]) * z / cam["fy"], z], 1).astype(np.float32)
    verts[V - 20:] = verts[:20]   # ties
    depth = rng.uniform(z0 - 1.2 * tau, z0 + spread + 1.2 * tau, (H, W)).astype(np.float32)
    depth[rng.random((H, W)) < 0.1] = 0.0
    want = oracle.associate(cam, tau, verts, depth=depth, brute=True)
    assert 0 < (want >= 0).sum() < W * H
    trk = T.Tracker(tiny.body.model, cam, dict(tiny.params, tau=tau), tiny.theta0)
    try:
        for _ in range(3):
            T.track_dbg_set(trk.ctx, T.TRACK_BUF_VERTS, verts)
            T.track_dbg_set(trk.ctx, T.TRACK_BUF_DEPTH, depth)
            assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_ASSOCIATE) == 0
            got = T.track_dbg_get(trk.ctx, T.TRACK_BUF_ASSOC, (W * H,), np.int32)
            np.testing.assert_array_equal(got, want)
    finally:
        trk.close()
