"""The pose step's tree form on plans of many fronts: several fronts a wave on
one level, parent entries that gather the shares of dozens of children, up to
seven levels, and plans that just fit its LDS.  Each is checked to run the
tree form (one that does not fit would be solved, unnoticed, by the dense
form) and then as the other skeletons are."""
import numpy as np
import pytest

import synth
import test_gpu_pose_tree as tree

pytestmark = pytest.mark.gpu

# limbs (parent limb or -1 for the root's six joints, hinges in a row), then the fronts and levels they make
PLANS = {
    "many": ([(-1, 1)] * 20 + [(-1, 2)] * 20, 41, 2),
    "most": ([(-1, 1)] * 31 + [(-1, 2)] * 25, 57, 2),
    "four levels": ([(-1, 6)] + [(0, 1)] * 12 + [(-1, 5)] + [(13, 2)] * 3 + [(k, 3) for k in (14, 15, 16) for _ in (0, 1)], 24, 4),
    "seven levels": ([(-1, 4), (0, 1), (0, 1), (1, 1), (1, 1), (3, 1), (3, 2), (5, 1), (5, 1), (7, 1), (7, 2), (9, 1), (9, 2)], 13, 7),
    "just fits": ([(-1, 6), (0, 2), (0, 9), (2, 2), (2, 5), (3, 2), (5, 4), (5, 1), (4, 4)], 9, 5),
    "just fits, wide": ([(-1, 8), (0, 8), (0, 5), (-1, 4), (3, 6), (2, 5), (1, 5), (4, 5), (7, 5), (8, 4), (8, 4)], 10, 4),
}


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available()
    from paper_1711_07999_amd import track
    track.lib()
    return track


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("plan", list(PLANS))
def test_tree_step(T, monkeypatch, plan, fp64):
    limbs, fronts, levels = PLANS[plan]
    m, P, _ = tree._model(limbs, np.random.default_rng(len(plan)))
    trk = T.Tracker(m, synth.make_arm().camera, synth.default_params(P, 1, 0.05), np.zeros(P))
    try:
        got = T.track_dbg_get(trk.ctx, T.TRACK_BUF_SOLVE_PLAN, (5,), np.int32)
    finally:
        trk.close()
    print(f"[pose_tree] {plan}: tree form, fronts, levels, elements, words {got}", flush=True)
    assert got[0] == 1 and got[1] == fronts and got[2] == levels
    monkeypatch.setitem(tree.SKELETONS, plan, limbs)
    tree.test_tree_step(T, plan, fp64)
