"""SC2 weights at the edges of the 128 x 128 output tiles, on the dense and the bit-count path, and
with weights beyond the histogram bins a workgroup keeps in LDS, against the oracle (bit-exact)."""
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import check_taps, run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def indoor(n, ratio, seed, **kw):
    return synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=ratio, **kw), seed)


@pytest.mark.parametrize("cap", [0, T.TR_SC2_SPARSE_CAP_MAX])
@pytest.mark.parametrize("n", [33, 256, 257, 383, 384, 385, 513, 769, 1025])
def test_tile_edges(n, cap):
    p = indoor(n, 0.3, 500 + n)
    prm = T.make_params(0.1, 0.1, k1=60, k2=2)
    say(f"tile edges n={n} cap={cap}")
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=60, max_k2=2)
    try:
        t = T.tr_tuning_get(reg.h, n)
        t.sc2_sparse_cap = cap
        T.tr_tuning_set(reg.h, n, 1, t)
        r, mask = run_single(reg, torch, p.src, p.dst, prm)
        check_taps(reg, p.src, p.dst, prm, r, mask, label=f"n={n} cap={cap}")
    finally:
        reg.close()


@pytest.mark.parametrize("n", [8127, 8128, 8300])
def test_weights_past_the_lds_bins(n):
    # nearly every pair compatible: the heaviest weights are n - 2 and just below, on both sides of
    # the 8126 bins in LDS
    p = indoor(n, 0.999, 600 + n, sigma=0.0)
    prm = T.make_params(0.01, 0.01, k1=200, k2=2)
    say(f"heavy weights n={n}")
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=200, max_k2=2)
    try:
        r, mask = run_single(reg, torch, p.src, p.dst, prm)
        check_taps(reg, p.src, p.dst, prm, r, mask, label=f"heavy n={n}", dense=False)
    finally:
        reg.close()
