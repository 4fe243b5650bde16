"""Compatibility where rounding alone separates lengths by more than the threshold (scenes 10^8 to 10^13
times larger than tau, a few noise-free matches among outliers): bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import turboreg as T
from parity import run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def scene(n, rigid, scale, seed):
    """n matches in a cube, `rigid` of them an exact (up to float32) rigid copy."""
    g = np.random.default_rng(seed)
    X, Y = (g.random((n, 3)) * scale - scale / 2 for _ in range(2))
    Q, _ = np.linalg.qr(g.standard_normal((3, 3)))
    k = g.permutation(n)[:rigid]
    Y[k] = X[k] @ (Q * np.sign(np.linalg.det(Q))).T
    return X.astype(np.float32), Y.astype(np.float32)


def check(scale, tau, n=2000, rigid=60):
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=20, max_k2=2)
    try:
        for seed in range(2):
            X, Y = scene(n, rigid, scale, seed)
            say(f"scale {scale} tau {tau} seed {seed}")
            r, _ = run_single(reg, torch, X, Y, T.make_params(tau, max(tau, 0.1), k1=20, k2=2))
            Co, _, _, _ = oracle.compat(X, Y, tau)
            C = reg.debug(T.TR_TAP_C)
            assert np.array_equal(C, Co), f"{int((C != Co).sum())} entries of C differ, edges {int(Co.sum()) // 2}"
            assert r.n_edges == int(Co.sum()) // 2
    finally:
        reg.close()


@pytest.mark.parametrize("scale,tau", [(100.0, 1e-8), (1e4, 2e-6), (1e4, 1e-5), (1e6, 1e-4), (1e7, 1e-3), (1e7, 1e-6),
                                       (4e7, 0.05)])
def test_scene_far_larger_than_the_threshold(scale, tau):
    check(scale, tau)
