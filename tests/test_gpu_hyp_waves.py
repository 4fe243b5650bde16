"""Hypothesis items of a long list (two workgroups of four waves per CU) give what a single pair's (eight waves) give."""
import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("graph", [T.TR_GRAPH_O2, T.TR_GRAPH_SC2])
@pytest.mark.parametrize("k2", [1, 2, 3, 8])
def test_batch_equals_single_pairs(k2, graph):
    ns, k1 = [3, 40, 257, 1000, 700, 1500], 1001   # 251 items a pair, the last of one pivot
    say(f"k2={k2} graph={graph}")
    pairs = [synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=0.2), 30 + n) for n in ns]
    prm = T.make_params(0.1, 0.1, k1=k1, k2=k2, graph=graph)
    reg = T.Registrar(max_n=max(ns), max_batch=len(ns), max_k1=k1, max_k2=k2)
    try:
        src, dst = (to_dev(torch, np.concatenate([getattr(p, f) for p in pairs])) for f in ("src", "dst"))
        offs = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
        out, mask = reg.register_batch(src, dst, to_dev(torch, offs), prm, max_n=max(ns))
        torch.cuda.synchronize()
        got, masks = T.parse_results(out, len(ns)), mask.cpu().numpy()
        poses = [reg.debug(T.TR_TAP_POSES, b) for b in range(len(ns))]
        inl = [reg.debug(T.TR_TAP_IN, b) for b in range(len(ns))]
        for b, p in enumerate(pairs):
            o1, m1 = reg.register(to_dev(torch, p.src), to_dev(torch, p.dst), prm)
            torch.cuda.synchronize()
            assert bytes(T.parse_results(o1)[0]) == bytes(got[b]), f"record of pair {b}"
            assert np.array_equal(m1.cpu().numpy()[:ns[b]], masks[offs[b]:offs[b + 1]]), f"mask of pair {b}"
            assert np.array_equal(reg.debug(T.TR_TAP_IN, 0), inl[b]), f"inlier numbers of pair {b}"
            ok = inl[b] >= 0
            assert np.array_equal(reg.debug(T.TR_TAP_POSES, 0)[ok], poses[b][ok]), f"poses of pair {b}"
    finally:
        reg.close()
