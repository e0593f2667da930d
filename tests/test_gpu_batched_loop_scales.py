"""The batched loop with register-resident weights on numbers of any magnitude: reverse sweeps whose rows grow, fall, start
from nothing or are tiny or huge, step by step against float64, and tiny initial states.

Slopes are 1 (tanh, states of zero), V is the identity and c zero, so G = dZ = -2 Y / (N O) is what the targets say; the
input is the identity, so dWx holds Delta itself.  Bound: three bf16 numbers hold all 24 bits of state and matrix, whatever the
numbers beside them are, so a step's product is off by the rounding of sums of 256 terms, at most 2^-21 of
sum |Wh| |delta|, and by 2^-134 |Wh| where delta is below about 1e-33 (the 1e-42).  Errors of the steps add up along the
same recursion as the terms."""
import pytest
import torch

import paper_1211_5590_amd as rnn

pytestmark = pytest.mark.gpu

KINDS = ["steady", "tiny", "huge", "jump", "late_zeros", "falls", "grows", "rows", "zero_start", "steep"]


def targets(kind, T, B, H):
    g = torch.Generator().manual_seed(T + H)
    Y = torch.randn(T, B, H, generator=g)
    if kind == "tiny":
        Y *= 1e-20                           # (the products around the loop hold all bits down to 1e-33)
    elif kind == "huge":
        Y *= 1e8
    elif kind == "jump":                     # 10^9 fold from one step to the next
        Y[T // 2:] *= 1e-9
    elif kind == "late_zeros":
        Y[T // 2:] = 0.0
    elif kind == "falls":
        Y *= 4.0 ** -torch.arange(T - 1, -1, -1).clamp(max=18)[:, None, None]
    elif kind == "grows":
        Y *= 8.0 ** -torch.arange(T)[:, None, None].clamp(max=20).float()
    elif kind == "rows":
        Y *= 10.0 ** -torch.arange(0, 4 * B, 4)[None, :, None].float()
    elif kind == "zero_start":               # the first state of the sweep is zero, the next one tiny
        Y *= 1e-15
        Y[T - 1] = 0.0
    elif kind == "steep":                    # nothing but the last step's error, which falls about 2^10 fold per step
        Y[:T - 1] = 0.0
        Y *= 2.0 ** 30
    return Y


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("H", [193, 224, 255, 256])
def test_reverse_rows_of_any_course(H, kind):
    T, B = 12 if kind == "steep" else 23, 6
    N = T * B
    Y = targets(kind, T, B, H)
    g = torch.Generator().manual_seed(H)
    Wh = torch.randn(H, H, generator=g) * (0.3 / H ** 0.5) * (2.0 ** -8 if kind == "steep" else 1.0)
    p = dict(Wx=torch.zeros(H, N), Wh=Wh, b=torch.zeros(H), V=torch.eye(H), c=torch.zeros(H))
    p = {k: v.cuda() for k, v in p.items()}
    dims = rnn.Dims(N, H, H, T, B, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    assert rnn.rnn_recurrence_variant(dims) == "batch_mfma"
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.zeros(T + 1, B, H, device="cuda")
    X, loss, dh0 = torch.eye(N, device="cuda").view(T, B, N), torch.zeros(1, device="cuda"), torch.zeros(B, H, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_loss(dims, p, h, Y.cuda(), loss, ws)
    rnn.rnn_bptt(dims, p, X, Y.cuda(), h, None, grads, dh0, ws)
    got = grads["dWx"].t().reshape(T, B, H).cpu().double()
    G = ((0.0 - Y) * torch.tensor(2.0 / (N * H), dtype=torch.float32)).double()
    W, delta, err = Wh.double(), torch.zeros(B, H, dtype=torch.float64), torch.zeros(B, H, dtype=torch.float64)
    for t in range(T - 1, -1, -1):
        delta, mag = G[t] + delta @ W, delta.abs() @ W.abs()
        err = err @ W.abs() + 2.0 ** -21 * (mag + G[t].abs()) + 1e-42
        worst = float(((got[t] - delta).abs() / err).max())
        assert worst <= 1.0, (t, worst)
    assert float(((dh0.cpu().double() - delta @ W).abs() / (err @ W.abs() + 2.0 ** -21 * (delta.abs() @ W.abs()) + 1e-42)).max()) <= 1.0


@pytest.mark.parametrize("exponent", [0, -20, -40, -60])
@pytest.mark.parametrize("H", [40, 193, 256])
def test_small_initial_states(H, exponent):
    """A state next to nothing against weights as much larger: the step's product is what it is at ordinary sizes.  Its bound is
    that of the reverse sweep; tanh adds its own rounding, which is that of numbers near one: a few 2^-24."""
    T, B = 2, 6
    g = torch.Generator().manual_seed(H)
    h0 = torch.randn(B, H, generator=g) * 2.0 ** exponent
    Wh = torch.randn(H, H, generator=g) * (0.5 / H ** 0.5) * 2.0 ** -exponent
    p = dict(Wx=torch.zeros(H, 2), Wh=Wh, b=torch.zeros(H), V=torch.zeros(H, 2), c=torch.zeros(2))
    p = {k: v.cuda() for k, v in p.items()}
    dims = rnn.Dims(2, H, 2, T, B, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    assert rnn.rnn_recurrence_variant(dims) == "batch_mfma"
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    hist = torch.zeros(T + 1, B, H, device="cuda")
    rnn.rnn_forward(dims, p, torch.zeros(T, B, 2, device="cuda"), h0.cuda(), hist, None, ws)
    ref = torch.tanh(h0.double() @ Wh.double().t())
    mag = h0.double().abs() @ Wh.double().abs().t()
    worst = float(((hist[1].cpu().double() - ref).abs() / (2.0 ** -21 * mag + 2.0 ** -22)).max())
    assert worst <= 1.0, worst
