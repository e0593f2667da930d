"""Products whose operands' leading dimension passes 2^26 (a vocabulary, or dense inputs, of tens of millions): lane
offsets of the ordinary tiles would not fit 32 bits there.  Every place such an operand has in the path -- K-contiguous
(U = X Wx^T, G = dZ V^T) and K-major (Z = H V, dV = H^T dZ, dWx = Delta^T X), with bias, overwriting and
accumulating -- against float64.

Bounds: an operand keeps 24 bits (16 with two parts).  A sum of 67 million terms of one sign is added up in parts
of at most 2^15 terms, 16 to a rounding: a part of 2048 roundings is off by 0.3 sqrt(2048 / 3) 2^-23 = 9e-7 of itself at most,
so 2e-6 for the whole; one after the other the terms would be off by sqrt(2^26 / 3) 0.3 2^-23 = 2e-4."""
import numpy as np
import pytest
import torch

import paper_1211_5590_amd as rnn

pytestmark = pytest.mark.gpu

WIDE = (1 << 26) + 37
CHUNK = 1 << 24


def chunks(n):
    return [(a, min(a + CHUNK, n)) for a in range(0, n, CHUNK)]


@pytest.mark.parametrize("flags", [0, rnn.FLAG_BF16X3_OUTPUT], ids=["three_parts", "two_parts"])
def test_a_wide_output_layer(flags):
    B, H, D, O = 3, 5, 4, WIDE
    g = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")   # noqa: E731
    # everything of one sign: Z - Y > 0, V > 0
    p = dict(Wx=rand(H, D) - 0.5, Wh=torch.eye(H, device="cuda"), b=rand(H) - 0.5, V=rand(H, O), c=rand(O))
    dims = rnn.Dims(D, H, O, 1, B, rnn.INPUT_DENSE, rnn.ACT_SIGMOID, rnn.LOSS_LINEAR_MSE, flags)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    X, Y = rand(1, B, D), -rand(1, B, O)
    h = torch.zeros(2, B, H, device="cuda")
    loss, dh0 = torch.zeros(1, device="cuda"), torch.zeros(B, H, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_forward(dims, p, X, None, h, None, ws)
    rnn.rnn_loss(dims, p, h, Y, loss, ws)
    rnn.rnn_bptt(dims, p, X, Y, h, None, grads, dh0, ws)
    torch.cuda.synchronize()
    h1 = h[1].double()
    eps = (256.0 if flags else 1.0) * 2.0 ** -24
    G, total = torch.zeros(B, H, dtype=torch.float64, device="cuda"), 0.0
    for a, z in chunks(O):
        V = p["V"][:, a:z].double()
        err = h1 @ V + p["c"][a:z].double() - Y[0, :, a:z].double()
        total += float(err.square().sum())
        dz = err * (2.0 / (B * O))
        G += dz @ V.t()
        dv = h1.t() @ dz
        assert float(((grads["dV"][:, a:z].double() - dv).abs() / dv).max()) <= 32 * eps, a
        assert float(((grads["dc"][a:z].double() - dz.sum(0)).abs() / dz.sum(0)).max()) <= 32 * eps, a
    assert abs(float(loss) - total / (B * O)) <= 1e-4 * total / (B * O)
    delta = G * h1 * (1 - h1)                            # Wh is the identity: dh0 is Delta itself
    worst = float(((dh0.double() - delta).abs() / delta).max())
    print("relative error of G", worst)
    assert worst <= 512 * eps if flags else worst <= 2e-6
    first = grads["dV"][:, -5000:].clone()
    dims.flags |= rnn.FLAG_ACCUMULATE | rnn.FLAG_BPTT_RECOMPUTE
    rnn.rnn_bptt(dims, p, X, Y, h, None, grads, dh0, ws)
    torch.cuda.synchronize()
    assert float(((grads["dV"][:, -5000:] - 2 * first).abs() / first).max()) <= 1e-6


def test_wide_dense_inputs():
    B, H, D, O = 3, 5, WIDE, 4
    g = torch.Generator(device="cuda").manual_seed(2)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")   # noqa: E731
    X = rand(1, B, D)
    p = dict(Wx=rand(H, D) * (3.0 / D), Wh=torch.eye(H, device="cuda"), b=rand(H) - 1.0, V=rand(H, O), c=rand(O))
    dims = rnn.Dims(D, H, O, 1, B, rnn.INPUT_DENSE, rnn.ACT_SIGMOID, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    Y = -rand(1, B, O)
    h = torch.zeros(2, B, H, device="cuda")
    loss, dh0 = torch.zeros(1, device="cuda"), torch.zeros(B, H, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_forward(dims, p, X, None, h, None, ws)
    rnn.rnn_loss(dims, p, h, Y, loss, ws)
    rnn.rnn_bptt(dims, p, X, Y, h, None, grads, dh0, ws)
    torch.cuda.synchronize()
    a = p["b"].double().expand(B, H).clone()
    for i, z in chunks(D):
        a += X[0, :, i:z].double() @ p["Wx"][:, i:z].double().t()
    # slope of the sigmoid at most 1/4; |a| up to 2.5; its own error 2^-22
    assert float((h[1].double() - torch.sigmoid(a)).abs().max()) <= 0.25 * 2.5 * 2e-6 + 2.0 ** -22
    delta = dh0.double()                                  # Wh is the identity
    for i, z in chunks(D):
        ref = delta.t() @ X[0, :, i:z].double()
        mag = delta.abs().t() @ X[0, :, i:z].double()
        assert float(((grads["dWx"][:, i:z].double() - ref).abs() / mag).max()) <= 16 * 2.0 ** -24, i
    assert float(loss) == float(loss) and np.isfinite(float(loss))
