"""Pivot collection at the edges of its 64-row by 64-column segments and of the sizes that deal them differently,
with few and with many keys per item and with ties that overflow the pool, against the oracle."""
import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import check_taps, run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k1", [3, 1000, 2500])
@pytest.mark.parametrize("n", [3, 63, 64, 65, 511, 512, 513, 1024, 1025, 1089, 2113])
def test_scan_edges(n, k1):
    say(f"scan n={n} k1={k1}")
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=0.3), 70 + n)
    prm = T.make_params(0.1, 0.1, k1=k1, k2=2)
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=2500, max_k2=2)
    try:
        r, mask = run_single(reg, torch, p.src, p.dst, prm)
        check_taps(reg, p.src, p.dst, prm, r, mask, label=f"n={n} k1={k1}")
    finally:
        reg.close()


@pytest.mark.parametrize("n", [300, 900, 1500])
def test_a_cluster_of_pivots_and_pool_overflow(n):
    # `block` matches in a row are one rigid copy: their segments hold nearly all pivots (more keys than an item
    # stages), all of one weight (a tie that overflows the pool at the larger size)
    rng = np.random.default_rng(n)
    block = n // 2
    X = ((rng.random((n, 3)) - 0.5) * 3.0).astype(np.float32)
    Y = ((rng.random((n, 3)) - 0.5) * 3.0).astype(np.float32)
    Y[64:64 + block] = X[64:64 + block] + np.float32(0.5)
    for k1 in (50, 1500):
        say(f"cluster n={n} k1={k1}")
        prm = T.make_params(0.01, 0.1, k1=k1, k2=2)
        reg = T.Registrar(max_n=n, max_batch=1, max_k1=1500, max_k2=2)
        try:
            r, mask = run_single(reg, torch, X, Y, prm)
            check_taps(reg, X, Y, prm, r, mask, label=f"cluster n={n} k1={k1}")
        finally:
            reg.close()


@pytest.mark.parametrize("ratio", [0.0, 0.3])
@pytest.mark.parametrize("n", [3, 257, 2049, 4100, 8192, 8193])
def test_single_pair_finds_the_batch_threshold(n, ratio):
    # a single pair's row scan finds the threshold itself up to 8192 matches, a batch's and a larger one's are given it
    say(f"threshold n={n} ratio={ratio}")
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=ratio), 90 + n)
    prm = T.make_params(0.1, 0.1, k1=300, k2=2)
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=300, max_k2=2)
    try:
        src, dst = torch.from_numpy(p.src).cuda(), torch.from_numpy(p.dst).cuda()
        offs = torch.tensor([0, n], dtype=torch.int32, device="cuda")
        got = []
        for batch in (False, True):
            out, mask = reg.register_batch(src, dst, offs, prm, max_n=n) if batch else reg.register(src, dst, prm)
            torch.cuda.synchronize()
            got.append((out.cpu().numpy().tobytes(), mask.cpu().numpy()[:n].tobytes(), reg.debug(T.TR_TAP_PIVOTS, 0).tobytes()))
        assert got[0] == got[1]
    finally:
        reg.close()
