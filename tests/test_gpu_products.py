"""The batched float32 products (three-way bf16 split on the matrix cores) at tile edges, remainders of
K and unaligned operands, through one-step dense calls: U = X Wx^T (both operands K-contiguous),
Z = H V, dV = H^T dZ and dWx = Delta^T X (K-major), against float64 from the call's own states.

Bound: every operand keeps its 24 bits, the dropped product terms are below 2^-24 |a b|, and a sum of K
terms is rounded about K/8 times, so |error| <= (2^-23 + sqrt(K/8) 2^-24) sum |a b|; the test allows twice
sqrt(K/8) + 4 units of 2^-24 sum |a b| (the factor covers the epilogue's own roundings)."""
import numpy as np
import pytest
import torch

import paper_1211_5590_amd as rnn

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1, 1), (5, 3, 2, 7), (63, 65, 17, 64), (129, 128, 15, 31), (257, 255, 33, 65), (256, 256, 48, 256),
         (700, 200, 513, 129), (4099, 513, 130, 2001)]   # rows, hidden, inputs, outputs


def close(name, got, ref, mag, K):
    bound = 2.0 * (np.sqrt(K / 8.0) + 4.0) * 2.0 ** -24 * mag + 1e-30
    worst = float(((got.double() - ref).abs() / bound).max())
    assert worst <= 1.0, (name, worst)


@pytest.mark.parametrize("flags", [0, rnn.FLAG_BF16X3_OUTPUT], ids=["three_parts", "two_parts"])
@pytest.mark.parametrize("N,H,D,O", SIZES)
def test_products_keep_float32_accuracy(N, H, D, O, flags):
    g = torch.Generator(device="cuda").manual_seed(N + H)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1   # noqa: E731
    X = torch.empty(N * D + 1, device="cuda")[1:].view(1, N, D)            # inputs are 4-byte aligned only
    X.copy_(rand(1, N, D))
    Y = rand(1, N, O)
    p = dict(Wx=rand(H, D) * 0.05, Wh=rand(H, H), b=rand(H), V=rand(H, O), c=rand(O))
    dims = rnn.Dims(D, H, O, 1, N, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, flags)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.zeros(2, N, H, device="cuda")
    loss = torch.zeros(1, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_forward(dims, p, X, None, h, None, ws)
    rnn.rnn_loss(dims, p, h, Y, loss, ws)
    rnn.rnn_bptt(dims, p, X, Y, h, None, grads, None, ws)
    torch.cuda.synchronize()
    x, h1, q = X[0].double(), h[1].double(), {k: v.double() for k, v in p.items()}
    # U enters through tanh (slope <= 1, rounded to float32)
    a = x @ q["Wx"].t() + q["b"]
    mag = x.abs() @ q["Wx"].abs().t() + q["b"].abs()
    close("h", h[1], torch.tanh(a), mag + 4.0, D)
    eps = 1.0 if not flags else 256.0          # two parts keep 16 bits of every operand
    scale = 2.0 / (N * O)
    dZ = (h1 @ q["V"] + q["c"] - Y[0].double()) * scale
    zmag = (h1.abs() @ q["V"].abs() + 2.0) * scale
    close("dV", grads["dV"], h1.t() @ dZ, eps * (h1.abs().t() @ (dZ.abs() + zmag)), N + H)
    D1 = (dZ @ q["V"].t()) * (1 - h1 * h1)
    dmag = (zmag @ q["V"].abs().t())
    close("dWx", grads["dWx"], D1.t() @ x, eps * 2.0 * (dmag.t() @ x.abs()), N + H + O)


def test_values_that_do_not_split_give_what_float32_gives():
    """Infinities, NaNs, values whose bf16 rounding overflows, and products that overflow."""
    N, H, D = 70, 130, 40
    g = torch.Generator(device="cpu").manual_seed(3)
    X = torch.rand(1, N, D, generator=g) - 0.5
    W = torch.rand(H, D, generator=g) - 0.5
    X[0, 3, 5], X[0, 4, 6], X[0, 9, 0], X[0, 20, 39], X[0, 69, 1] = float("inf"), float("-inf"), 3.4e38, float("nan"), 1e38
    W[7, 1], W[11, 5] = 1e30, 0.0
    p = dict(Wx=W.cuda(), Wh=torch.zeros(H, H, device="cuda"), b=torch.zeros(H, device="cuda"),
             V=torch.zeros(H, 3, device="cuda"), c=torch.zeros(3, device="cuda"))
    dims = rnn.Dims(D, H, 3, 1, N, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.zeros(2, N, H, device="cuda")
    rnn.rnn_forward(dims, p, X.cuda(), None, h, None, ws)
    got = h[1].cpu()
    ref = torch.tanh(X[0] @ W.t())
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    fine = ~torch.isnan(ref)
    assert float((got[fine] - ref[fine]).abs().max()) < 1e-5
