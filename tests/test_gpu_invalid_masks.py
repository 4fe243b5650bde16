"""Mask entries of pairs with fewer than three matches: cleared, whatever the buffer held, in batches below and
above the size from which pairs are ordered."""
import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ns", [[300, 2, 64, 1, 0, 3], [1], [2, 400, 1] * 7 + [0]])
def test_masks_of_tiny_pairs(ns):
    base = synth.CONFIGS["indoor_n1000"]
    pairs = [synth.make_pair(base.replace(n=max(n, 3), inlier_ratio=0.5), 50 + k) for k, n in enumerate(ns)]
    src, dst = (to_dev(torch, np.concatenate([getattr(p, f)[:n] for p, n in zip(pairs, ns)])) for f in ("src", "dst"))
    offs = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    reg = T.Registrar(max_n=400, max_batch=len(ns), max_k1=50, max_k2=2)
    try:
        prm = T.make_params(0.1, 0.1, k1=50, k2=2)
        say(f"{len(ns)} pairs")
        masks = torch.full((int(offs[-1]),), 0xA5, dtype=torch.uint8, device="cuda")
        out, _ = reg.register_batch(src, dst, to_dev(torch, offs), prm, max_n=400, masks=masks)
        torch.cuda.synchronize()
        m = masks.cpu().numpy()
        for b, r in enumerate(T.parse_results(out, len(ns))):
            own = m[offs[b]:offs[b + 1]]
            if ns[b] < 3:
                assert r.status == T.TR_ERR_INVALID_ARG and not own.any(), b
            else:
                assert r.status != T.TR_ERR_INVALID_ARG and own.max(initial=0) <= 1 and int(own.sum()) == max(r.best_inliers, 0), b
    finally:
        reg.close()
