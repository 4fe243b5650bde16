"""Scorer gradients at the edges of the training kernel's steps (32 samples per wave, 128 per workgroup,
32768 per pass of 256 workgroups) against a float64 pass with bfloat16 weights and activations.

Tolerance: an activation may round to the neighbouring bfloat16 (2^-8 relative), which moves a gradient
by at most about twice that; float32 rounding is far below."""
import math

import numpy as np
import pytest

from paper_2507_01439_amd import train_scorer
from paper_2507_01439_amd import turboreg as T

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
TOL = 2.0 ** -7


@pytest.fixture(scope="module")
def reg():
    r = T.Registrar(max_n=64, max_batch=1, max_k1=1, max_k2=1)
    w = train_scorer.init_params(3)
    w[1216:1280] = np.linspace(-0.3, 0.3, 64)   # layer biases that need all their float32 bits
    w[5376:5440] = np.linspace(0.2, -0.4, 64)
    w[5504] = 0.123456
    T.tr_scorer_set(r.h, w)
    yield r, torch.from_numpy(w)
    r.close()


def samples(m, seed):
    g = np.random.default_rng(seed)
    return (torch.from_numpy(g.random((m, 19), dtype=np.float32) * 2 - 0.5).to(torch.bfloat16),
            torch.from_numpy((g.random(m) < 0.3).astype(np.uint8)))


def reference(w, f, y):
    def bf(v):
        return v.to(torch.bfloat16).double()

    W1, b1 = bf(w[:1216]).view(64, 19), w[1216:1280].double()
    W2, b2 = bf(w[1280:5376]).view(64, 64), w[5376:5440].double()
    W3, b3 = bf(w[5440:5504]), w[5504].double()
    c = math.sqrt(2 / math.pi)

    def gelu(v):
        th = torch.tanh(c * (v + 0.044715 * v ** 3))
        return bf((0.5 * v * (1 + th)).float()), 0.5 * (1 + th) + 0.5 * v * (1 - th * th) * c * (1 + 3 * 0.044715 * v * v)

    x = f.double()
    a1, g1 = gelu(x @ W1.T + b1)
    a2, g2 = gelu(a1 @ W2.T + b2)
    s = a2 @ W3 + b3
    ds = (torch.sigmoid(s) - y.double()) / len(y)
    d2 = ds[:, None] * W3 * g2
    d1 = (d2 @ W2) * g1
    loss = torch.nn.functional.binary_cross_entropy_with_logits(s, y.double())
    return [d1.T @ x, d1.sum(0), d2.T @ a1, d2.sum(0), a2.T @ ds, ds.sum()[None]], loss


def grads(reg, feat, lab):
    g = torch.full((T.TR_MLP_NPARAM,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    T.tr_mlp_grads(reg.h, feat, lab, lab.shape[0], g, loss)
    torch.cuda.synchronize()
    return g.cpu(), loss.cpu()


@pytest.mark.parametrize("m", [1, 2, 31, 32, 33, 127, 128, 129, 1000, 32768, 32769, 40007])
def test_gradients(reg, m):
    print(f"gradients m={m}", flush=True)
    r, w = reg
    f, y = samples(m, m)
    g, loss = grads(r, f.view(torch.int16).cuda(), y.cuda())
    ref, lref = reference(w, f, y)
    at = 0
    for t in ref:
        got = g[at:at + t.numel()].double().view(t.shape)
        at += t.numel()
        assert float((got - t).norm()) <= TOL * float(t.norm()) + 1e-12, (m, at)
    assert abs(float(loss[0]) - float(lref)) <= TOL * float(lref)


def test_unaligned_slice_and_repeat(reg):
    # rows of a feature table start on two-byte boundaries; the sums do not depend on the call
    r, _ = reg
    f, y = samples(1501, 9)
    table, lab = f.view(torch.int16).cuda(), y.cuda()
    a, la = grads(r, table[1:], lab[1:])
    b, lb = grads(r, table[1:].clone(), lab[1:].clone())
    c, lc = grads(r, table[1:], lab[1:])
    assert torch.equal(a, b) and torch.equal(a, c) and torch.equal(la, lb) and torch.equal(la, lc)
