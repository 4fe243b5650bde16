"""Scorer gradients of hidden units far to the left of zero: GELU and its derivative are 0 there, whatever the
size of the value, so such units pass nothing back."""
import numpy as np
import pytest

from paper_2507_01439_amd import turboreg as T
from test_gpu_train_tiles import grads, reference

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
TOL = 2.0 ** -7   # an activation may round to the neighbouring bfloat16


def params():
    """Unit 0 of layer 1 is -x0 and unit 1 is x0; unit 0 of layer 2 is -(unit 1); the rest is small."""
    g = np.random.default_rng(8)
    w = np.zeros(T.TR_MLP_NPARAM, np.float32)
    W1, W2 = w[:1216].reshape(64, 19), w[1280:5376].reshape(64, 64)
    W1[2:, 1:] = g.standard_normal((62, 18)) * 0.3
    W1[0, 0], W1[1, 0] = -1.0, 1.0
    W2[:, 2:] = g.standard_normal((64, 62)) * 0.2
    W2[0, 1] = -1.0
    W2[:, 0] = 0.5
    w[5440:5504] = g.standard_normal(64) * 0.3
    return w


@pytest.mark.parametrize("big", [1.0, 9.0, 14.0, 30.0, 1e4, 1e11, 1e13, 1e15, 1e18])
def test_gradients_of_saturated_units(big):
    print(f"pre-activation -{big}", flush=True)
    w = params()
    g = np.random.default_rng(9)
    f = g.random((70, 19), dtype=np.float32)
    f[:, 0] = 0
    f[[3, 40, 69], 0] = big
    f, y = torch.from_numpy(f).to(torch.bfloat16), torch.from_numpy((g.random(70) < 0.4).astype(np.uint8))
    reg = T.Registrar(max_n=64, max_batch=1, max_k1=1, max_k2=1)
    try:
        T.tr_scorer_set(reg.h, w)
        got, loss = grads(reg, f.view(torch.int16).cuda(), y.cuda())
    finally:
        reg.close()
    ref, lref = reference(torch.from_numpy(w), f, y)
    assert abs(float(loss[0]) - float(lref)) <= TOL * float(lref)
    at = 0
    for t in ref:
        v = got[at:at + t.numel()].double().view(t.shape)
        at += t.numel()
        assert torch.isfinite(v).all()
        # a tensor row by row: one row (unit 1's share of dW2) may be as large as `big`
        v, t = (v, t) if t.dim() == 2 else (v[:, None], t[:, None])
        bound = TOL * t.norm(dim=1) + 1e-6
        assert bool(((v - t).norm(dim=1) <= bound).all()), (at, float(((v - t).norm(dim=1) / bound).max()))
