"""Scorer gradients to float32 accuracy: on samples whose activations stay clear of bfloat16 ties (so that both
sides round them alike) every gradient tensor agrees with a float64 pass to 2^-19 of its norm.

The tolerance is 32 float32 roundings of one sign. Deltas of 16 bits instead of 24 (the last of the three
bfloat16 terms of a delta left out) miss it: the test plants that in the float64 pass and sees it fail."""
import numpy as np
import pytest

from test_gpu_train_tiles import grads, reference, reg  # noqa: F401 (reg is the fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
TOL = 2.0 ** -19


def clear_of_ties(w, f):
    """Samples none of whose activations lies within 2^-16 relative of the middle of two bfloat16 values."""
    def bf(v):
        return v.to(torch.bfloat16).double()

    def clear(a):
        u = (a.float().view(torch.int32) & 0xFFFF) - 0x8000   # 2^-24 relative each, 0 at a tie
        return ((u.abs() > 2 ** 8) | (a == 0)).all(1)

    def gelu(v):
        return 0.5 * v * (1 + torch.tanh((2 / np.pi) ** 0.5 * (v + 0.044715 * v ** 3)))

    a1 = gelu(f.double() @ bf(w[:1216]).view(64, 19).T + w[1216:1280].double())
    a2 = gelu(bf(a1.float()) @ bf(w[1280:5376]).view(64, 64).T + w[5376:5440].double())
    return clear(a1) & clear(a2)


def narrow_deltas(w, f, y):
    """The reference with layer 2's deltas cut to 16 bits (their first two bfloat16 terms): dW2 alone."""
    def bf(v):
        return v.to(torch.bfloat16).double()

    c = (2 / np.pi) ** 0.5

    def gelu(v):
        th = torch.tanh(c * (v + 0.044715 * v ** 3))
        return bf((0.5 * v * (1 + th)).float()), 0.5 * (1 + th) + 0.5 * v * (1 - th * th) * c * (1 + 3 * 0.044715 * v * v)

    a1, _ = gelu(f.double() @ bf(w[:1216]).view(64, 19).T + w[1216:1280].double())
    a2, g2 = gelu(a1 @ bf(w[1280:5376]).view(64, 64).T + w[5376:5440].double())
    s = a2 @ bf(w[5440:5504]) + w[5504].double()
    d2 = ((torch.sigmoid(s) - y.double()) / len(y))[:, None] * bf(w[5440:5504]) * g2
    cut = (d2.float().view(torch.int32) & ~0xFF).view(torch.float32).double()
    return cut.T @ a1


@pytest.mark.parametrize("m", [33, 129, 4000])
def test_gradients_keep_float32(reg, m):   # noqa: F811
    r, w = reg
    g = np.random.default_rng(100 + m)
    f = torch.from_numpy(g.random((8 * m, 19), dtype=np.float32) * 2 - 0.5).to(torch.bfloat16)
    f = f[clear_of_ties(w, f)][:m].contiguous()
    assert f.shape[0] == m
    y = torch.from_numpy((g.random(m) < 0.3).astype(np.uint8))
    ref, lref = reference(w, f, y)
    assert float((narrow_deltas(w, f, y) - ref[2]).norm()) > 2 * TOL * float(ref[2].norm())
    print(f"gradients m={m}", flush=True)
    got, loss = grads(r, f.view(torch.int16).cuda(), y.cuda())
    at = 0
    for t in ref:
        v = got[at:at + t.numel()].double().view(t.shape)
        at += t.numel()
        err = float((v - t).norm()) / float(t.norm())
        print(f"  {tuple(t.shape)}: {err:.2e}", flush=True)
        assert err <= TOL, (m, at, err)
    assert abs(float(loss[0]) - float(lref)) <= TOL * float(lref)
