"""The normal equations over the column lists of their workgroups: lists that
just fill a block of 16 or start the next, all 128 columns, chunks with two
and with no vertices observed, more chunks than workgroups (a workgroup's
chunks then touch different columns), and one, two and four influences."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# mesh sampling (vertices a ring, rings), hinges per limb, a vertex' limb
# changes every so many vertices, influences
CASES = {
    "16": ((16, 8), [9], 1, 1),
    "17": ((16, 8), [10], 1, 2),
    "32": ((37, 54), [13, 12], 1, 1),
    "33": ((37, 54), [13, 13], 1, 4),
    "128": ((37, 54), [3] * 40 + [1], 1, 1),
    "chunks": ((257, 257), [9] * 13, 128, 1),
    "chunks-blended": ((257, 257), [5] * 13, 128, 2),
}


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


def _model(ring, limbs, every, infl, rng):
    m = dict(synth.make_arm(*ring).model)
    parent, kind, tips = [k - 1 for k in range(6)], [1] * 3 + [0] * 3, []
    for n in limbs:
        parent += [5] + list(range(len(parent), len(parent) + n - 1))
        kind += [0] * n
        tips.append(len(parent) - 1)
    P, V = len(parent), m["rest_xyz"].shape[0]
    axis = rng.normal(size=(P, 3))
    axis[:6] = np.tile(np.eye(3), (2, 1))
    offset = np.zeros((P, 7), np.float32)
    offset[:, 0] = 1.0
    offset[:, 4:] = rng.normal(0, 0.05, (P, 3))
    m.update(joint_parent=np.array(parent, np.int32), joint_type=np.array(kind, np.int32),
             joint_axis=(axis / np.linalg.norm(axis, axis=1)[:, None]).astype(np.float32), joint_offset=offset,
             link_joint=np.array([5] + tips, np.int32))
    first = 1 + np.arange(V) // every % len(limbs)
    m["skin_link"] = np.full((V, 4), -1, np.int32)
    m["skin_w"] = np.zeros((V, 4), np.float32)
    for k in range(infl):
        m["skin_link"][:, k] = (first + k) % (len(tips) + 1)
        m["skin_w"][:, k] = 2.0 ** -(k + 1 if k + 1 < infl else k)
    return m, P, V


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("case", list(CASES))
def test_gram_matches_the_oracle(T, case, mode):
    """Float32 rows carry about 1e-6 of a generator's lever arm, some 1e-5 of
    a column's norm, and the split forms' products 2^-17: each entry is within
    1e-4 of the product of its columns' norms.  Entries of columns that no
    vertex touches together are exactly zero in both."""
    ring, limbs, every, infl = CASES[case]
    rng = np.random.default_rng(infl + len(limbs))
    m, P, V = _model(ring, limbs, every, infl, rng)
    print(f"[gram] {case} P={P} V={V} mode={mode}", flush=True)
    th = rng.uniform(-0.1, 0.1, P)
    phi = rng.normal(0, 0.002, (V, 3)).astype(np.float32)
    v32 = oracle.skin(m, th, phi.astype(np.float64))[0].astype(np.float32)
    n = rng.normal(size=(V, 3))
    n32 = (n / np.linalg.norm(n, axis=1)[:, None]).astype(np.float32)
    delta = rng.normal(0, 0.01, (V, 3)).astype(np.float32)
    cnt = rng.integers(0, 4, V).astype(np.int32)
    cnt[np.arange(V) // 128 % 5 == 3] = 0
    cnt[(np.arange(V) // 128 % 5 == 1) & (np.arange(V) % 128 > 1)] = 0
    trk = T.Tracker(m, synth.make_arm().camera, dict(synth.default_params(P, 1, 0.05), gram_mode=mode), th)
    try:
        for buf, arr in ((T.TRACK_BUF_THETA, th), (T.TRACK_BUF_PHI, phi), (T.TRACK_BUF_VERTS, v32),
                         (T.TRACK_BUF_NORMALS, n32), (T.TRACK_BUF_COUNT, cnt), (T.TRACK_BUF_DELTA, delta)):
            T.track_dbg_set(trk.ctx, buf, arr)
        assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_NORMAL_EQ) == 0
        G = T.track_dbg_get(trk.ctx, T.TRACK_BUF_GRAM, (P + 1, P + 1), np.float64)
    finally:
        trk.close()
    ps = oracle.pose_system(m, th, phi.astype(np.float64), n32.astype(np.float64), delta.astype(np.float64), cnt)
    Jr = np.concatenate([ps["J"], ps["r"][:, None]], 1)
    want, nrm = Jr.T @ Jr, np.linalg.norm(Jr, axis=0)
    np.testing.assert_array_equal(G, G.T)
    assert (np.abs(G[:P, P] - ps["b"]) <= 1e-4 * nrm[:P] * nrm[P] + 1e-12).all()
    assert (np.abs(G - want) <= 1e-4 * np.outer(nrm, nrm) + 1e-12).all()
    touch = np.abs(ps["J"]) > 0
    apart = (touch.astype(np.float32).T @ touch.astype(np.float32)) == 0
    assert (G[:P, :P][apart] == 0.0).all()


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_many_workgroups_equal_few(T, mode):
    """Three streams of 345 chunks in one server's launch take workgroups of
    half the waves: the same pose and offsets bit for bit as each alone."""
    body = synth.make_arm(210, 210)
    m, cam, P, V = body.model, body.camera, len(body.model["joint_parent"]), body.model["rest_xyz"].shape[0]
    assert 3 * (-(-V // 128)) > 1024 >= -(-V // 128)
    prm = dict(synth.default_params(P, 2, 0.05), gram_mode=mode, active=None)
    rng = np.random.default_rng(5)
    ths = [np.where(body.angular, rng.uniform(-0.1, 0.1, P), rng.uniform(-0.01, 0.01, P)) for _ in range(3)]
    frames = [synth.render_frame(m, cam, synth.pose_surface(m, 0.8 * th), rng, 0.0, 0.0) for th in ths]
    print(f"[gram] 3 x {V} vertices mode={mode}", flush=True)
    alone = []
    for th, d in zip(ths, frames):
        trk = T.Tracker(m, cam, dict(prm, active=np.ones(P, np.uint8)), th)
        try:
            assert trk.frame(d) == 0, T.track_last_error()
            alone.append(trk.state()[:2])
        finally:
            trk.close()
    sv = T.track_server_create(prm, 1 << 36, 8)
    try:
        ids = [T.track_server_open(sv, m, cam, th) for th in ths]
        for k, d in enumerate(frames):
            T.track_server_submit(sv, ids[k], d, tag=k)
        done = []
        for _ in range(20):
            if len(done) == 3:
                break
            T.track_server_step(sv)
            done += T.track_server_poll(sv)
        assert len(done) == 3 and all(c["status"] == 0 for c in done)
        for k in range(3):
            th, phi = T.track_server_state(sv, ids[k], P, V)
            assert np.array_equal(th, alone[k][0]) and np.array_equal(phi, alone[k][1]), k
    finally:
        T.track_server_destroy(sv)
