"""SC2 tiles counted bit by bit at every tile edge (256 .. 1024), in one pass over the rows and in several,
beside tiles left to the matrix cores, for single pairs, ragged batches, the automatic rule of large pairs,
the SC2 graph and the learned features: every weight, row statistic and record equals the dense run's."""
import hashlib

import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# batch, largest n, inlier ratio; tile edges on 256 CUs: 256, 512, 768, 768 and 1024
CASES = [(1, 1500, 0.3), (1, 9000, 0.02), (24, 2700, 0.1), (64, 2100, 0.02), (1, 16500, 0.01)]


def run(B, n, ratio, cap, mode):
    ns = [n] if B == 1 else [max(1, n - 97 * k % n) for k in range(B)]
    base = synth.CONFIGS["indoor_n1000"]
    pairs = [synth.make_pair(base.replace(n=v, inlier_ratio=ratio), 900 + k % 4) for k, v in enumerate(ns)]
    prm = T.make_params(0.1, 0.1, k1=200, k2=2, graph=T.TR_GRAPH_SC2 if mode == "sc2" else T.TR_GRAPH_O2,
                        pivot_mode=T.TR_PIVOTS_LEARNED if mode == "learned" else T.TR_PIVOTS_PLAIN)
    reg = T.Registrar(max_n=n, max_batch=B, max_k1=200, max_k2=2)
    try:
        t = T.tr_tuning_get(reg.h, n, B)
        t.sc2_sparse_cap = cap
        T.tr_tuning_set(reg.h, n, B, t)
        T.tr_scorer_set(reg.h, np.random.default_rng(3).standard_normal(5505).astype(np.float32) * 0.2)
        src, dst = (to_dev(torch, np.concatenate([getattr(p, f) for p in pairs])) for f in ("src", "dst"))
        offs = to_dev(torch, np.concatenate([[0], np.cumsum(ns)]).astype(np.int32))
        got = {}
        for _ in range(2):   # the second call finds the first one's counters and weights
            out, mask = reg.register(src, dst, prm) if B == 1 else reg.register_batch(src, dst, offs, prm, max_n=n)
            torch.cuda.synchronize()
        got["records"], got["masks"] = out.cpu().numpy().tobytes(), mask.cpu().numpy().tobytes()
        for b in sorted({0, B // 2, B - 1}):
            got[f"weights {b}"] = hashlib.sha256(np.triu(reg.debug(T.TR_TAP_G, b), 1).tobytes()).digest()
        if mode == "learned":
            pool = reg.debug(T.TR_TAP_PLAIN_PIVOTS, 0)[:, :2]   # only the pool's endpoints are scored
            got["pool"] = pool.tobytes()
            got["scores"] = reg.debug(T.TR_TAP_SCORES, 0)[np.unique(pool[pool >= 0])].tobytes()
            feat = torch.zeros((sum(ns), 19), dtype=torch.int16, device="cuda")
            T.tr_features_batch(reg.h, src, dst, offs, B, n, prm, feat)
            torch.cuda.synchronize()
            got["features"] = feat.cpu().numpy().tobytes()
        return got
    finally:
        reg.close()


@pytest.mark.parametrize("mode", ["o2", "sc2", "learned"])
@pytest.mark.parametrize("B,n,ratio", CASES)
def test_bit_counts_equal_the_dense_product(B, n, ratio, mode):
    say(f"B={B} n={n} {mode}")
    want = run(B, n, ratio, 1, mode)   # nearly every tile on the matrix cores
    for cap in (0, 256, T.TR_SC2_SPARSE_CAP_MAX):
        say(f"  cap={cap}")
        got = run(B, n, ratio, cap, mode)
        for key in want:
            assert got[key] == want[key], f"cap={cap}: {key} differ"
