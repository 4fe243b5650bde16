"""Pivots per hypothesis work item: the counts the dispatch picks for few pivots and several cliques each
(one, two or four per item), on both graphs and with the error-based ranking, against the oracle."""
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import check_taps, run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def reg():
    r = T.Registrar(max_n=1100, max_batch=1, max_k1=600, max_k2=8)
    yield r
    r.close()


@pytest.mark.parametrize("graph", [T.TR_GRAPH_O2, T.TR_GRAPH_SC2])
@pytest.mark.parametrize("k1,k2", [(1, 8), (3, 3), (17, 5), (130, 8), (255, 3), (257, 4), (600, 5)])
def test_items(reg, k1, k2, graph):
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=1100 if graph else 450, inlier_ratio=0.3), 40 + k1 + k2)
    prm = T.make_params(0.1, 0.1, k1=k1, k2=k2, graph=graph)
    say(f"items k1={k1} k2={k2} graph={graph}")
    r, mask = run_single(reg, torch, p.src, p.dst, prm)
    check_taps(reg, p.src, p.dst, prm, r, mask, label=f"k1={k1} k2={k2} graph={graph}")


@pytest.mark.parametrize("flag", [T.TR_FLAG_RANK_MAE, T.TR_FLAG_RANK_MSE])
def test_ranked_scores_do_not_depend_on_the_item(reg, flag):
    # 8 cliques of 9 pivots, one pivot per item: every pose scores the bits tr_score_poses gives it
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=700, inlier_ratio=0.3), 77)
    say("ranked items")
    run_single(reg, torch, p.src, p.dst, T.make_params(0.1, 0.1, k1=9, k2=8, flags=flag))
    poses, inl, sc = (reg.debug(t) for t in (T.TR_TAP_POSES, T.TR_TAP_IN, T.TR_TAP_RANK_SCORES))
    i2 = torch.zeros(72, dtype=torch.int32, device="cuda")
    s2 = torch.zeros(72, dtype=torch.float32, device="cuda")
    T.tr_score_poses(reg.h, torch.from_numpy(p.src).cuda(), torch.from_numpy(p.dst).cuda(), 700,
                     torch.from_numpy(poses).cuda(), 72, 0.1, 1 if flag == T.TR_FLAG_RANK_MAE else 2, i2, s2)
    torch.cuda.synchronize()
    ok = inl >= 0
    assert ok.any() and (i2.cpu().numpy()[ok] == inl[ok]).all() and (s2.cpu().numpy()[ok] == sc[ok]).all()
