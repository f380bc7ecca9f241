"""The surrogate's products at ragged batches: rows that do not fill a 64-row tile,
a last k-step that is not whole, one or several splits of the weight gradients, and
weights that are not 16-byte aligned (scalar fetches), forward and backward.

Reference: the same network in float64 on the bf16-rounded weights with every layer's
activations and gradients rounded to bf16 where the kernels do.  What is left are
float32 sums of at most 12,000 terms (relative 1e-5 or so) and bf16 roundings that
such a difference tips over (a few of a million, 2^-8 each): 2e-3 of a tensor's norm."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _bf(x):
    return x.to(torch.float32).to(torch.bfloat16).double()


def _reference(W, b, x, t):
    a, zs, acts = _bf(x), [], [_bf(x)]
    for k in range(4):
        z = a @ W[k] + b[k]
        zs.append(z)
        if k < 3:
            a = _bf(torch.nn.functional.silu(z))
            acts.append(a)
    B = len(x)
    g = 2 * (zs[3] - t.double()) / (3 * B)
    dW, db = [None] * 4, [None] * 4
    loss = ((zs[3] - t.double()) ** 2).mean()
    for k in range(3, -1, -1):
        db[k] = g.sum(0)
        dW[k] = acts[k].T @ _bf(g)
        if k:
            s = torch.sigmoid(zs[k - 1])
            g = (_bf(g) @ W[k].T) * s * (1 + zs[k - 1] * (1 - s))
    return zs[3], loss, dW, db


@pytest.mark.parametrize("batch", [1, 3, 63, 64, 65, 255, 256, 257, 1000, 4099])
@pytest.mark.parametrize("shift", [0, 1])
def test_forward_and_gradients(batch, shift):
    from paper_2607_25585_amd import _ffi, surrogate as S
    torch.manual_seed(batch)
    print("case batch", batch, "shift", shift, flush=True)
    m = S.MLP(seed=3)
    m.p[m.nw:] = 0.1 * torch.randn(m.nb, device="cuda")
    if shift:  # weights one element off a 16-byte boundary
        pb = torch.empty(m.nw + 1, dtype=torch.bfloat16, device="cuda")
        pb[1:] = m.pb
        m.pb = pb[1:]
    x, t = torch.randn(batch, 7, device="cuda"), torch.randn(batch, 3, device="cuda")
    W, o = [], 0
    for fi, fo in zip(S.LAYERS[:-1], S.LAYERS[1:]):
        W.append(m.pb[o:o + fi * fo].double().view(fi, fo))
        o += fi * fo
    b, o = [], m.nw
    for fo in S.LAYERS[1:]:
        b.append(m.p[o:o + fo].double())
        o += fo
    y, loss, dW, db = _reference(W, b, x, t)
    got_y = m.forward(x).double()
    got_loss = float(m.gradients(x, t))
    near = lambda got, want: float(torch.linalg.vector_norm(got - want)) <= 2e-3 * float(torch.linalg.vector_norm(want))  # noqa: E731
    assert near(got_y, y)
    assert abs(got_loss - float(loss)) <= 2e-3 * float(loss)
    o = 0
    for k, (fi, fo) in enumerate(zip(S.LAYERS[:-1], S.LAYERS[1:])):
        assert near(m.g[o:o + fi * fo].double().view(fi, fo), dW[k]), ("dW", k)
        o += fi * fo
    for k, fo in enumerate(S.LAYERS[1:]):
        assert near(m.g[o:o + fo].double(), db[k]), ("db", k)
        o += fo
    assert ctypes.sizeof(_ffi.FtlmMlpWeights) == 64
