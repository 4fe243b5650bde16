"""Training features at the edges of the row blocks (64 rows, 64- and 128-column blocks), with duplicate
and non-finite points and bins at exact edges, against the oracle (bit-exact)."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def want(X, Y, tau):
    Co, _, _, _ = oracle.compat(X, Y, tau)
    F = oracle.features(X, Y, tau, Co, oracle.sc2(Co))
    u = F.astype(np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) & 0xFFFF).astype(np.uint16)


def run(pairs, tau):
    ns = [p[0].shape[0] for p in pairs]
    offs = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    reg = T.Registrar(max_n=max(ns), max_batch=len(ns), max_k1=1, max_k2=1)
    try:
        feat = torch.zeros((int(offs[-1]), 19), dtype=torch.int16, device="cuda")
        T.tr_features_batch(reg.h, torch.from_numpy(np.concatenate([p[0] for p in pairs])).cuda(),
                            torch.from_numpy(np.concatenate([p[1] for p in pairs])).cuda(),
                            torch.from_numpy(offs).cuda(), len(ns), max(ns), T.make_params(tau, tau, 1, 1), feat)
        torch.cuda.synchronize()
        got = feat.cpu().numpy().view(np.uint16)
        return [got[offs[k]:offs[k + 1]] for k in range(len(ns))], [reg.debug(T.TR_TAP_C, k) for k in range(len(ns))]
    finally:
        reg.close()


def test_row_block_edges():
    pairs = []
    for n in (3, 63, 64, 65, 127, 128, 129, 257, 640, 1000):
        p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=0.4), 700 + n)
        pairs.append((p.src, p.dst))
    say("feature rows at block edges")
    got, C = run(pairs, 0.1)
    for k, (X, Y) in enumerate(pairs):
        assert np.array_equal(C[k], oracle.compat(X, Y, 0.1)[0]), X.shape
        assert np.array_equal(got[k], want(X, Y, 0.1)), X.shape


def test_exact_edges_and_duplicates():
    # points on a lattice: length differences fall exactly on bin edges; repeated points; tau 1, edges k / 4
    g = np.random.default_rng(3)
    X = g.integers(-4, 5, size=(300, 3)).astype(np.float32) * 0.25
    Y = g.integers(-4, 5, size=(300, 3)).astype(np.float32) * 0.25
    Y[:, 1:] = X[:, 1:]
    X[50:60], Y[50:60] = X[0], Y[0]
    say("feature bins at exact edges")
    got, C = run([(X, Y)], 1.0)
    assert np.array_equal(C[0], oracle.compat(X, Y, 1.0)[0])
    assert np.array_equal(got[0], want(X, Y, 1.0))
