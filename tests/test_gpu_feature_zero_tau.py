"""Training features at thresholds whose bin width is zero, against the oracle (bit-exact)."""
import numpy as np
import pytest

import oracle
from paper_2507_01439_amd import synth
from parity import say
from test_gpu_feature_rows import run, want

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tau", [0.0, 1e-45, 1e-38])   # bin width 0, 0 (underflow) and subnormal
def test_every_bin_edge_at_zero(tau):
    # a match's other matches all fall into the last bin (those at a NaN distance into the first), and the
    # match itself into none
    pairs = []
    for n in (3, 64, 65, 300):
        p = synth.make_pair(synth.CONFIGS["indoor_n1000"].replace(n=n, inlier_ratio=0.4), 800 + n)
        pairs.append((p.src.copy(), p.dst.copy()))
    for cloud in pairs[3]:
        cloud[10:14] = cloud[10]
    pairs[3][0][100, 1] = np.inf
    pairs[3][1][200, 0] = np.nan
    say(f"features at tau={tau}")
    got, C = run(pairs, tau)
    for k, (X, Y) in enumerate(pairs):
        assert np.array_equal(C[k], oracle.compat(X, Y, tau)[0]), X.shape
        assert np.array_equal(got[k], want(X, Y, tau)), X.shape
