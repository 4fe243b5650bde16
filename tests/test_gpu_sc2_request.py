"""The SC2 path on request: sc2_sparse_cap = 0 asks for the dense product of every tile at any size, and is kept
as asked; groups never set use bit counts beyond 8192 matches. The path changes no result."""
import numpy as np
import pytest

from paper_2507_01439_amd import synth
from paper_2507_01439_amd import turboreg as T
from parity import run_single, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,ratio", [(8192, 0.1), (8193, 0.02), (12000, 0.02)])
def test_the_product_on_request(n, ratio, tmp_path):
    p = synth.make_pair(synth.CONFIGS["outdoor_n20000"].replace(n=n, inlier_ratio=ratio), synth.pair_seed(6, 40))
    prm = T.make_params(0.6, 0.6, k1=300, k2=2)
    reg = T.Registrar(max_n=n, max_batch=1, max_k1=300, max_k2=2)
    try:
        default = T.tr_tuning_get(reg.h, n, 1)
        assert default.sc2_sparse_cap == (0 if n <= 8192 else 2048)
        say(f"n={n} default")
        got = [run_single(reg, torch, p.src, p.dst, prm)]
        for cap in (0, 2048):
            default.sc2_sparse_cap = cap
            T.tr_tuning_set(reg.h, n, 1, default)
            say(f"n={n} cap={cap}")
            got.append(run_single(reg, torch, p.src, p.dst, prm))
            assert T.tr_tuning_get(reg.h, n, 1).sc2_sparse_cap == cap
            path = str(tmp_path / f"tuning{cap}.txt")
            T.tr_tuning_save(reg.h, path)
            assert open(path).read().split()[-1] == str(cap)
        for r, m in got[1:]:
            assert bytes(r) == bytes(got[0][0]) and np.array_equal(m, got[0][1])
    finally:
        reg.close()
