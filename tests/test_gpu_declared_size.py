"""Batches whose declared max_n is far above their pairs: every record, mask, weight and feature is that of the
same batch declared at its own size, with and without requested bit counts, in pairs few, many and mixed."""
import hashlib

import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def run(pairs, declared, cap, learned):
    ns = [p.src.shape[0] for p in pairs]
    B = len(ns)
    reg = T.Registrar(max_n=declared, max_batch=B, max_k1=100, max_k2=2)
    try:
        if cap is not None:
            t = T.tr_tuning_get(reg.h, declared, B)
            t.sc2_sparse_cap = cap
            T.tr_tuning_set(reg.h, declared, B, t)
        T.tr_scorer_set(reg.h, np.random.default_rng(3).standard_normal(5505).astype(np.float32) * 0.2)
        src, dst = (to_dev(torch, np.concatenate([getattr(p, f) for p in pairs])) for f in ("src", "dst"))
        offs = to_dev(torch, np.concatenate([[0], np.cumsum(ns)]).astype(np.int32))
        prm = T.make_params(0.6, 0.6, k1=100, k2=2,
                            pivot_mode=T.TR_PIVOTS_LEARNED if learned else T.TR_PIVOTS_PLAIN)
        for _ in range(2):   # the second call finds the first one's counters and weights
            out, mask = reg.register_batch(src, dst, offs, prm, max_n=declared)
            torch.cuda.synchronize()
        got = {"records": out.cpu().numpy().tobytes(), "masks": mask.cpu().numpy().tobytes()}
        for b in sorted({0, B // 2, B - 1}):
            got[f"weights {b}"] = hashlib.sha256(np.triu(reg.debug(T.TR_TAP_G, b), 1).tobytes()).digest()
        feat = torch.zeros((sum(ns), 19), dtype=torch.int16, device="cuda")
        T.tr_features_batch(reg.h, src, dst, offs, B, declared, prm, feat)
        torch.cuda.synchronize()
        got["features"] = feat.cpu().numpy().tobytes()
        return got
    finally:
        reg.close()


@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("ns,declared", [([1000] * 5, 9000), ([300, 257, 3, 700], 8192), ([130] * 300, 2000),
                                         ([2300, 800, 64] * 8, 10000), ([8300] + [600] * 7, 12000),
                                         # compatibility lists of 80, 360, 810 and 5400 tiles: 8, 16, 32, 128 rows
                                         ([300] * 8, 8192), ([1000] * 10, 5000), ([500] * 81, 3000),
                                         ([1000] * 150, 2000)])
def test_results_do_not_depend_on_the_declared_size(ns, declared, learned):
    base = synth.CONFIGS["outdoor_n20000"]
    pairs = [synth.make_pair(base.replace(n=n, inlier_ratio=0.1), 300 + k % 5) for k, n in enumerate(ns)]
    say(f"{len(ns)} pairs of up to {max(ns)}, own size")
    want = run(pairs, max(ns), 0, learned)
    for cap in (None, 0, T.TR_SC2_SPARSE_CAP_MAX):
        say(f"  declared {declared}, limit {cap}")
        got = run(pairs, declared, cap, learned)
        for key in want:
            assert got[key] == want[key], (cap, key)
