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



def same_numbers(got, ref, tol, name):
    """NaN where the reference is, the same infinities, and the finite values within tol of the largest of them."""
    got, ref = got.cpu().double(), ref.double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref)), (name, int(torch.isnan(got).sum()), int(torch.isnan(ref).sum()))
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(got), inf) and torch.equal(got[inf], ref[inf]), name
    fine = torch.isfinite(ref)
    if fine.any():
        assert float((got[fine] - ref[fine]).abs().max()) <= tol * float(ref[fine].abs().max()), name


# rows, hidden, inputs: which form U = X Wx^T takes
FORMS_U = {"tile_64": (70, 130, 40), "tile_128": (2500, 2500, 37), "tile_256": (4096, 4096, 260), "k_cut": (64, 64, 4096)}


@pytest.mark.parametrize("kind", ["nan", "mixed"])
@pytest.mark.parametrize("form", list(FORMS_U))
def test_values_that_do_not_split_in_both_k_contiguous_operands(form, kind):
    """NaNs alone are left to the split products, anything else has the tile computed again in float32; either way the
    results that do not meet such a value are what they are without it."""
    N, H, D = FORMS_U[form]
    g = torch.Generator().manual_seed(N + H)
    X = (torch.rand(N, D, generator=g) - 0.5) * 0.2
    W = torch.rand(H, D, generator=g) - 0.5
    nan, inf = float("nan"), float("inf")
    X[3, 5], X[N - 1, D - 1], W[H - 2, 7] = nan, nan, nan
    if kind == "mixed":
        X[5, 0], X[6, D - 1], X[7, 1], W[11, 2], W[H - 1, D - 2] = inf, -inf, 3.4e38, inf, -3.4e38
        W[:, 1] *= 1e-3                       # 3.4e38 times it stays finite
        X[:, D - 2] *= 1e-3
    p = dict(Wx=W.cuda(), Wh=torch.zeros(H, H, device="cuda"), b=torch.zeros(H, device="cuda"),
             V=torch.zeros(H, 3, device="cuda"), c=torch.zeros(3, device="cuda"))
    dims = rnn.Dims(D, H, 3, 1, N, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.zeros(2, N, H, device="cuda")
    rnn.rnn_forward(dims, p, X.cuda().view(1, N, D), None, h, None, ws)
    same_numbers(h[1], torch.tanh(X.double() @ W.double().t()), 1e-5, form)


# rows, hidden, outputs
FORMS_DV = {"tile_64": (60, 70, 90), "tile_128": (300, 2500, 2500), "tile_256": (260, 4096, 4096), "k_cut": (4096, 64, 64)}


@pytest.mark.parametrize("flags", [0, rnn.FLAG_BF16X3_OUTPUT], ids=["three_parts", "two_parts"])
@pytest.mark.parametrize("kind", ["nan", "mixed"])
@pytest.mark.parametrize("form", list(FORMS_DV))
def test_values_that_do_not_split_in_the_backward_products(form, kind, flags):
    """dV = H^T dZ (both operands K-major), G = dZ V^T and the logits H V, through targets that are not finite."""
    N, H, O = FORMS_DV[form]
    g = torch.Generator().manual_seed(N + O)
    rand = lambda *s: torch.rand(*s, generator=g) - 0.5   # noqa: E731
    hrow, Y = rand(N, H), rand(N, O)
    nan, inf = float("nan"), float("inf")
    Y[3, O - 1], Y[N - 1, 0] = nan, nan
    if kind == "mixed":
        Y[4, 3], Y[5, 3], Y[6, O - 2] = inf, inf, -inf
        hrow[4, 9] = 0.0                      # 0 times infinity
    p = dict(Wx=torch.zeros(H, 2), Wh=rand(H, H) / H, b=torch.zeros(H), V=rand(H, O), c=rand(O))
    p = {k: v.cuda() for k, v in p.items()}
    dims = rnn.Dims(2, H, O, 1, N, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, flags)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.zeros(2, N, H, device="cuda")
    h[1] = hrow.cuda()
    X, Yd = torch.zeros(1, N, 2, device="cuda"), Y.cuda().view(1, N, O)
    loss, dh0 = torch.zeros(1, device="cuda"), torch.zeros(N, H, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_loss(dims, p, h, Yd, loss, ws)
    rnn.rnn_bptt(dims, p, X, Yd, h, None, grads, dh0, ws)
    torch.cuda.synchronize()
    h64, V = hrow.double(), p["V"].cpu().double()
    dZ = (h64 @ V + p["c"].cpu().double() - Y.double()) * (2.0 / (N * O))
    tol = 2e-4 if flags else 1e-5
    same_numbers(grads["dV"], h64.t() @ dZ, tol, "dV")
    odd = ~torch.isfinite(dZ).all(1)
    delta = (dZ[~odd] @ V.t()) * (1 - h64[~odd] ** 2)
    got = dh0.cpu().double()
    assert not torch.isfinite(got[odd]).any()
    ref = delta @ p["Wh"].cpu().double()
    assert float((got[~odd] - ref).abs().max()) <= tol * float(ref.abs().max())


@pytest.mark.parametrize("flags", [0, rnn.FLAG_BF16X3_OUTPUT], ids=["three_parts", "two_parts"])
@pytest.mark.parametrize("N,H,O", [(90, 70, 200), (700, 200, 10000), (4096, 260, 4096)], ids=["tile_64", "tile_128", "tile_256"])
def test_row_statistics_of_a_tile_that_is_computed_again(N, H, O, flags):
    """A state of 3.4e38 against weights of about 1e-38: the logits are ordinary numbers, though it does not split."""
    g = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") - 0.5   # noqa: E731
    h = torch.zeros(2, N, H, device="cuda")
    h[1] = rand(N, H)
    p = dict(Wx=rand(O, H), Wh=rand(H, H) / H, b=rand(H), V=rand(H, O), c=rand(O))
    h[1, :, 4] *= 1e-3
    h[1, 7, 4], h[1, N - 1, 4] = 3.4e38, -3.4e38
    p["V"][4] *= 1e-38
    dims = rnn.Dims(O, H, O, 1, N, rnn.INPUT_TOKENS, rnn.ACT_TANH, rnn.LOSS_SOFTMAX_CE, flags)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    y = torch.randint(0, O, (1, N), generator=g, device="cuda", dtype=torch.int32)
    loss = torch.zeros(1, device="cuda")
    rnn.rnn_loss(dims, p, h, y, loss, ws)
    z = h[1].double() @ p["V"].double() + p["c"].double()
    want = float((torch.logsumexp(z, 1) - z.gather(1, y[0].long()[:, None])[:, 0]).mean())
    assert abs(float(loss) - want) <= 1e-4 * abs(want)


def test_a_nan_does_not_slow_the_products_down():
    """NaNs are looked for once more where a tile shows them, no more: a training run that has diverged keeps its pace (1.3
    times the time of finite numbers; computing the tiles again wavefront by wavefront took 10 times)."""
    N, H, O = 4096, 1024, 4096
    g = torch.Generator(device="cuda").manual_seed(8)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") - 0.5   # noqa: E731
    h = torch.zeros(2, N, H, device="cuda")
    h[1] = rand(N, H)
    p = dict(Wx=rand(8, H), Wh=rand(H, H) / H, b=rand(H), V=rand(H, O), c=rand(O))
    dims = rnn.Dims(8, H, O, 1, N, rnn.INPUT_TOKENS, rnn.ACT_TANH, rnn.LOSS_SOFTMAX_CE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    x = torch.zeros(1, N, device="cuda", dtype=torch.int32)
    y = torch.randint(0, O, (1, N), generator=g, device="cuda", dtype=torch.int32)
    loss = torch.zeros(1, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best():
        times = []
        for _ in range(5):
            t0.record()
            rnn.rnn_loss(dims, p, h, y, loss, ws)
            rnn.rnn_bptt(dims, p, x, y, h, None, grads, None, ws)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)
    finite = best()
    h[1, 5, 3] = float("nan")
    spoilt = best()
    print(f"finite {finite:.3f} ms, with a NaN {spoilt:.3f} ms")
    assert spoilt < 3.0 * finite
