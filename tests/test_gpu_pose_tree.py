"""The pose step's tree form on skeletons that put its fronts at the edges of
what the kernel distinguishes: rows that just fill a register width or start
the next, one pivot under many later rows, one front alone, more fronts than
waves with all of their shares in one parent entry, several levels."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# limbs (parent limb or -1 for the root's six joints, hinges in a row)
SKELETONS = {
    "one": [(-1, 1)],
    "widths": [(-1, n) for n in (1, 2, 9, 10, 17, 18, 24, 25)],
    "many": [(-1, 1)] * 31 + [(-1, 3)] * 30,
    "deep": [(-1, 20)] + [(0, 1)] * 25 + [(-1, 8)] + [(26, 2)] * 3 + [(k, 4) for k in (27, 28, 29) for _ in range(2)],
}


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


def _model(limbs, rng):
    """The small arm's mesh on another skeleton: a link at each limb's tip,
    every vertex on one link."""
    m = dict(synth.make_arm().model)
    parent, kind, tips = [k - 1 for k in range(6)], [1] * 3 + [0] * 3, []
    for up, n in limbs:
        at = 5 if up < 0 else tips[up]
        for _ in range(n):
            parent.append(at)
            kind.append(0)
            at = len(parent) - 1
        tips.append(at)
    P, V = len(parent), m["rest_xyz"].shape[0]
    axis = rng.normal(size=(P, 3))
    axis[:6] = np.tile(np.eye(3), (2, 1))
    offset = np.zeros((P, 7), np.float32)
    offset[:, 0] = 1.0
    offset[:, 4:] = rng.normal(0, 0.05, (P, 3))
    m.update(joint_parent=np.array(parent, np.int32), joint_type=np.array(kind, np.int32),
             joint_axis=(axis / np.linalg.norm(axis, axis=1)[:, None]).astype(np.float32), joint_offset=offset,
             link_joint=np.array([5] + tips, np.int32))
    m["skin_link"] = np.full_like(m["skin_link"], -1)
    m["skin_link"][:, 0] = np.arange(V) % (len(tips) + 1)
    m["skin_w"] = np.zeros_like(m["skin_w"])
    m["skin_w"][:, 0] = 1.0
    return m, P, V


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("skeleton", list(SKELETONS))
def test_tree_step(T, skeleton, fp64):
    """The step equals the oracle's solve of the GPU's own Gram matrix.  A
    Cholesky solve's backward error is at most (3 P + 1) u |R^T| |R|, whose
    entries are at most one once the damped matrix has a unit diagonal, and
    the factor's rows hold few of them: so the scaled step is compared to
    (3 P + 3) u kappa, kappa the scaled matrix's condition number (at most
    P + 1 with a damping of 1), two u more for the rounded input."""
    rng = np.random.default_rng(len(skeleton))
    m, P, V = _model(SKELETONS[skeleton], rng)
    print(f"[pose_tree] {skeleton} P={P} fp64={fp64}", flush=True)
    cam = synth.make_arm().camera
    prm = dict(synth.default_params(P, 1, 0.05, lambda_k=1.0), pose_solve_fp64=fp64)
    th = rng.uniform(-0.1, 0.1, P)
    n = rng.normal(size=(V, 3))
    trk = T.Tracker(m, cam, prm, th)
    try:
        for buf, arr in ((T.TRACK_BUF_THETA, th),
                         (T.TRACK_BUF_VERTS, (m["rest_xyz"] + rng.normal(0, 0.1, (V, 3))).astype(np.float32)),
                         (T.TRACK_BUF_NORMALS, (n / np.linalg.norm(n, axis=1)[:, None]).astype(np.float32)),
                         (T.TRACK_BUF_COUNT, rng.integers(0, 4, V).astype(np.int32)),
                         (T.TRACK_BUF_DELTA, rng.normal(0, 0.01, (V, 3)).astype(np.float32))):
            T.track_dbg_set(trk.ctx, buf, arr)
        assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_NORMAL_EQ) == 0
        G = T.track_dbg_get(trk.ctx, T.TRACK_BUF_GRAM, (P + 1, P + 1), np.float64)
        assert T.track_dbg_run(trk.ctx, T.TRACK_PASS_POSE_STEP) == 0
        step = T.track_dbg_get(trk.ctx, T.TRACK_BUF_STEP, (P,), np.float64)
        th_new = T.track_dbg_get(trk.ctx, T.TRACK_BUF_THETA, (P,), np.float64)
    finally:
        trk.close()
    x = oracle.lm_solve(G[:P, :P], G[:P, P], 1.0)
    d = np.sqrt(2.0 * np.diag(G)[:P])
    A = np.triu(G[:P, :P]) / np.outer(d, d)
    kappa = np.linalg.cond(A + np.triu(A, 1).T + 0.5 * np.eye(P))
    u = np.finfo(np.float64 if fp64 else np.float32).eps / 2
    err, tol = np.linalg.norm(d * (step - x)) / np.linalg.norm(d * x), (3 * P + 3) * u * kappa
    print(f"  scaled step difference {err:.2e}, bound {tol:.2e}, kappa {kappa:.1f}", flush=True)
    assert np.linalg.norm(x) > 0 and err <= tol
    np.testing.assert_allclose(th_new, th - step, rtol=0, atol=1e-15)
