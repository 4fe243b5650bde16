"""The compatibility kernel's guarded decisions against the oracle (bit-exact) where the guard works
hardest: thresholds far below, near and above the scene's extent, far-off and huge coordinates,
duplicate points, and the row counts per work item that the list length selects."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def check(X, Y, tau, label):
    n = X.shape[0]
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=20, max_k2=2)
    try:
        say(label)
        r, _ = run_single(reg, torch, X, Y, T.make_params(tau, max(tau, 0.1), k1=20, k2=2))
        Co, b32, _, _ = oracle.compat(X, Y, tau)
        C = reg.debug(T.TR_TAP_C)
        assert np.array_equal(C, Co), f"{label}: C differs at {np.argwhere(C != Co)[:5].tolist()}"
        assert r.n_boundary_pairs == b32 and r.n_edges == int(Co.sum()) // 2, label
    finally:
        reg.close()


def pair(n, seed, ratio=0.3, scale=1.0, shift=0.0):
    p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=ratio), seed)
    return ((p.src * np.float32(scale) + np.float32(shift)).astype(np.float32),
            (p.dst * np.float32(scale) - np.float32(shift)).astype(np.float32))


@pytest.mark.parametrize("tau", [0.0, 1e-12, 1e-6, 1e-3, 0.1, 0.7, 3.0, 50.0, 1e9])
def test_thresholds(tau):
    X, Y = pair(420, 11)
    check(X, Y, tau, f"tau={tau}")


@pytest.mark.parametrize("scale,shift,tau", [(1e-4, 0.0, 1e-5), (40.0, 0.0, 0.01), (1.0, 3e4, 0.1), (1e4, 1e6, 50.0),
                                             (1e9, 0.0, 1e8), (1e19, 0.0, 1e17), (1e-20, 0.0, 1e-21)])
def test_coordinate_ranges(scale, shift, tau):
    X, Y = pair(333, 12, scale=scale, shift=shift)
    check(X, Y, tau, f"scale={scale} shift={shift} tau={tau}")


def test_duplicates_and_nonfinite():
    X, Y = pair(300, 13)
    X[40:80], Y[40:60] = X[7], Y[7]            # coincident in both clouds, or in one
    X[100] = X[101] = (np.inf, 0, 0)
    Y[102, 1], X[150, 2] = np.nan, -np.inf
    check(X, Y, 0.1, "duplicates, infinities, NaN")


@pytest.mark.parametrize("n", [2000, 3100, 8500])
def test_rows_per_item(n):
    # lists of 136, 325 and 2278 tiles: 8, 16 and 32 rows per item (batches cover the longer ones)
    X, Y = pair(n, 14 + n, ratio=0.1)
    check(X, Y, 0.1, f"n={n}")


@pytest.mark.parametrize("B", [64])
def test_long_lists(B):
    # 64 pairs of up to 1500 matches: 4992 tiles, 128 rows per item
    rng = np.random.default_rng(5)
    ns = rng.integers(1200, 1501, size=B)
    ps = [pair(int(n), 900 + k) for k, n in enumerate(ns)]
    offs = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    reg = T.Registrar(max_n=1500, max_batch=B, max_k1=20, max_k2=2)
    try:
        say("64 pairs, 128 rows per item")
        out, _ = reg.register_batch(torch.from_numpy(np.concatenate([p[0] for p in ps])).cuda(),
                                    torch.from_numpy(np.concatenate([p[1] for p in ps])).cuda(),
                                    torch.from_numpy(offs).cuda(), T.make_params(0.1, 0.1, k1=20, k2=2))
        torch.cuda.synchronize()
        rs = T.parse_results(out, B)
        for k in range(0, B, 7):
            Co, b32, _, _ = oracle.compat(ps[k][0], ps[k][1], 0.1)
            assert np.array_equal(reg.debug(T.TR_TAP_C, k), Co), k
            assert rs[k].n_boundary_pairs == b32 and rs[k].n_edges == int(Co.sum()) // 2, k
    finally:
        reg.close()
