"""Caller-given poses scored at the edges of the workgroups' pose counts and of the match groups: inlier numbers
equal the oracle's, and a pose's bits do not depend on the poses beside it."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

THETA = 0.1


def poses_near(p, P, rng):
    t = p.t + rng.standard_normal((P, 3)) * 10.0 ** rng.uniform(-3, 0, (P, 1))
    return np.concatenate([np.tile(np.asarray(p.R).reshape(1, 9), (P, 1)), t], 1).astype(np.float32)


@pytest.mark.parametrize("metric", [0, 1, 2])
@pytest.mark.parametrize("n,P", [(1, 1), (63, 512), (257, 513), (1024, 514), (1025, 1024), (2049, 1025), (5000, 1027)])
def test_pose_scores(n, P, metric):
    say(f"n={n} P={P} metric={metric}")
    rng = np.random.default_rng(n + P)
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=0.3), 40 + n)
    poses = poses_near(p, P, rng)
    poses[P // 2] = np.nan   # scores nothing
    src, dst = to_dev(torch, p.src), to_dev(torch, p.dst)
    reg = T.Registrar(max_n=n + 2, max_batch=1, max_k1=8, max_k2=2)

    def score(ps):
        inl = torch.full((len(ps),), -1, dtype=torch.int32, device="cuda")
        sc = torch.full((len(ps),), -1.0, dtype=torch.float32, device="cuda")
        T.tr_score_poses(reg.h, src, dst, n, to_dev(torch, ps), len(ps), THETA, metric, inl, sc if metric else None)
        torch.cuda.synchronize()
        return inl.cpu().numpy(), sc.cpu().numpy()

    try:
        inl, sc = score(poses)
        ok = np.arange(P) != P // 2
        assert np.array_equal(inl[ok], oracle.score(p.src, p.dst, poses[ok], np.ones(ok.sum(), np.int32), THETA))
        assert inl[P // 2] == 0
        for a, b in ((0, 1), (P - 1, P), (P // 3, P // 3 + min(7, P - P // 3))):   # one pose a workgroup
            i1, s1 = score(poses[a:b])
            assert np.array_equal(i1, inl[a:b]) and s1.tobytes() == sc[a:b].tobytes()
        if metric:
            X, Y = p.src.astype(np.float64), p.dst.astype(np.float64)
            r = np.linalg.norm(np.einsum("pij,nj->pni", poses[ok, :9].reshape(-1, 3, 3).astype(np.float64), X)
                               + poses[ok, None, 9:] - Y, axis=2)
            c = np.maximum(1.0 - r / THETA, 0.0) ** metric
            # float32 residuals of metres err by up to 3e-6 m, a term by 2 x 3e-6 / 0.1 and its rounding
            tol = 1e-4 * (1.0 + inl[ok])
            assert (np.abs(sc[ok] - c.sum(1)) <= tol).all()
            assert sc[P // 2] == 0.0
    finally:
        reg.close()
