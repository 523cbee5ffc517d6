"""The association's search over its window and list sizes, bit-exact against
the oracle's exhaustive search: windows of one tile around a tile's own, of
exactly the two that come with the pixels, of rings beyond them and of the
whole image; images that end inside a tile; cells with none, one and more
vertices than a pass takes (from their regions, and from the overflow list
before a layout exists); duplicate vertices; pixels without a measurement
and pixels far behind the surface beside pixels on it."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# width, height, focal length, depth range, cutoff, pixels the vertices cover (None: the image and around it)
CASES = {
    "own tiles": (67, 43, 90.0, (2.9, 3.1), 0.1, None),
    "two tiles": (160, 120, 131.25, (1.1, 1.3), 0.1, None),
    "a third ring": (160, 117, 131.25, (0.55, 0.7), 0.1, None),
    "many rings": (131, 90, 131.25, (0.5, 0.9), 0.25, None),
    "whole image": (75, 50, 300.0, (0.4, 0.8), 0.5, None),
    "one tile of vertices": (160, 120, 131.25, (1.0, 1.02), 0.1, (40, 40, 46, 46)),
    "one cell of vertices": (40, 33, 90.0, (1.0, 1.3), 0.1, (20, 16, 22, 18)),
}


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


@pytest.mark.parametrize("case", list(CASES))
def test_windows_and_lists_are_bit_exact(T, tiny, case):
    W, H, f, (z0, z1), tau, box = CASES[case]
    print(f"[windows] {case}", flush=True)
    cam = dict(width=W, height=H, fx=f, fy=f * 1.01, cx=(W - 1) / 2.0, cy=(H - 1) / 2.0)
    V = tiny.body.model["rest_xyz"].shape[0]
    rng = np.random.default_rng(sorted(CASES).index(case))
    bu0, bv0, bu1, bv1 = box or (-4, -4, W + 4, H + 4)
    z = rng.uniform(z0, z1, V)
    u, v = rng.uniform(bu0, bu1, V), rng.uniform(bv0, bv1, V)
    verts = np.stack([(u - cam["cx"]) * z / cam["fx"], (v - cam["cy"]) * z / cam["fy"], z], 1).astype(np.float32)
    verts[V - 50:] = verts[:50]
    depth = rng.uniform(z0 - 0.5 * tau, z1 + 0.5 * tau, (H, W)).astype(np.float32)
    what = rng.random((H, W))
    depth[what < 0.15] = 0.0
    depth[(what >= 0.15) & (what < 0.30)] = z1 + 3 * tau
    depth[(what >= 0.30) & (what < 0.31)] = np.inf
    depth[(what >= 0.31) & (what < 0.32)] = np.nan
    depth[: H // 4, : W // 3] = z1 + 3 * tau   # whole tiles of background
    want = oracle.associate(cam, tau, verts, depth=depth, brute=True)
    assert 0 < (want >= 0).sum() < W * H
    trk = T.Tracker(tiny.body.model, cam, dict(tiny.params, tau=tau), tiny.theta0)
    try:
        T.track_dbg_set(trk.ctx, T.TRACK_BUF_VERTS, verts)
        T.track_dbg_set(trk.ctx, T.TRACK_BUF_DEPTH, depth)
        for _ in range(3):   # without a layout, then twice in the one the last left
            assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_ASSOCIATE) == 0
            got = T.track_dbg_get(trk.ctx, T.TRACK_BUF_ASSOC, (H * W,), np.int32)
            count = T.track_dbg_get(trk.ctx, T.TRACK_BUF_COUNT, (V,), np.uint32)
            np.testing.assert_array_equal(got, want)
            np.testing.assert_array_equal(count, np.bincount(want[want >= 0], minlength=V))
    finally:
        trk.close()
