"""Boundary counts at thresholds below the report's own band of 1e-6: equal to the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import turboreg as T
from parity import run_single, say
from test_gpu_compat_ratio import scene

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("scale,tau", [(0.1, 1e-9), (0.1, 1e-8), (0.1, 1e-7), (0.1, 1e-6), (0.3, 1e-7), (1.0, 2e-6),
                                       (100.0, 1e-8)])
def test_boundary_pairs_of_tiny_thresholds(scale, tau):
    n = 2000
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=20, max_k2=2)
    try:
        for seed in range(2):
            X, Y = scene(n, 60, scale, seed)
            say(f"scale {scale} tau {tau} seed {seed}")
            r, _ = run_single(reg, torch, X, Y, T.make_params(tau, 0.1, k1=20, k2=2))
            Co, b32, _, _ = oracle.compat(X, Y, tau)
            assert np.array_equal(reg.debug(T.TR_TAP_C), Co)
            assert r.n_boundary_pairs == b32, (r.n_boundary_pairs, b32)
    finally:
        reg.close()
