"""Classes that an output bias of minus infinity takes out (a padded or masked vocabulary): the loss stays
finite and the gradients of the other classes are those of the smaller vocabulary, however long the masked
stretch is and wherever it lies in the parts over which the row statistics are formed (32, 64 and 128
columns), in every form of the output layer.  Reference: float64 from the call's own states."""
import numpy as np
import pytest
import torch

import paper_1211_5590_amd as rnn

pytestmark = pytest.mark.gpu


def problem(H, O, T, B, masked, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *s, k=1.0: torch.randn(*s, generator=g, device="cuda") * k   # noqa: E731
    p = dict(Wx=normal(O, H, k=0.3), Wh=normal(H, H, k=0.3 / np.sqrt(H)), b=normal(H, k=0.1),
             V=normal(H, O, k=1.0 / np.sqrt(H)), c=normal(O, k=0.1))
    live = torch.ones(O, dtype=torch.bool, device="cuda")
    for a, z in masked:
        p["c"][a:z] = float("-inf")
        live[a:z] = False
    ids = torch.nonzero(live)[:, 0]
    x = ids[torch.randint(0, len(ids), (T * B + 1,), generator=g, device="cuda")].to(torch.int32)
    return p, live, x[:-1].contiguous(), x[1:].contiguous()


def check(p, live, y, h_rows, loss, grads):
    h, V, c = h_rows.double(), p["V"].double()[:, live], p["c"].double()[live]
    place = torch.cumsum(live, 0) - 1
    z = h @ V + c
    lse = torch.logsumexp(z, 1)
    t = place[y.long()]
    want = float((lse - z.gather(1, t[:, None])[:, 0]).mean())
    assert np.isfinite(float(loss)) and abs(float(loss) - want) <= 1e-4 * abs(want), (float(loss), want)
    dz = torch.exp(z - lse[:, None])
    dz[torch.arange(len(t), device="cuda"), t] -= 1.0
    dz /= len(t)
    for name, ref in (("dV", h.t() @ dz), ("dc", dz.sum(0))):
        got = grads[name].double()
        assert not got[..., ~live].any(), name
        assert float((got[..., live] - ref).abs().max()) <= 1e-3 * float(ref.abs().max()), name
    for name in ("dWx", "dWh", "db"):
        assert torch.isfinite(grads[name]).all(), name


def buffers(p, T, B, H):
    return (torch.zeros(T + 1, B, H, device="cuda"), torch.full((1,), float("nan"), device="cuda"),
            {"d" + k: torch.full_like(v, float("nan")) for k, v in p.items()})


# hidden, classes, steps, batch: which form of the logits product serves it
FORMS = {
    "tile_64": (68, 160, 36, 7),
    "tile_64_many_classes": (1024, 1024, 40, 8),
    "tile_64_uncut_many_classes": (340, 1024, 40, 8),
    "tile_128": (200, 10000, 35, 20),
    "tile_256": (260, 4096, 64, 64),
    "k_cut": (1024, 260, 11, 6),
    "short_sequence": (40, 640, 20, 1),
}


@pytest.mark.parametrize("where", ["tail", "head", "inside"])
@pytest.mark.parametrize("width", [31, 32, 64, 128])
@pytest.mark.parametrize("form", list(FORMS))
def test_three_calls(form, width, where):
    H, O, T, B = FORMS[form]
    a = {"tail": O - width, "head": 0, "inside": min(256, O - 160)}[where]
    for flags in (0, rnn.FLAG_BF16X3_OUTPUT):
        p, live, x, y = problem(H, O, T, B, [(a, a + width)], 31 * width + O)
        dims = rnn.Dims(O, H, O, T, B, rnn.INPUT_TOKENS, rnn.ACT_TANH, rnn.LOSS_SOFTMAX_CE, flags)
        h, loss, grads = buffers(p, T, B, H)
        ws = torch.full((rnn.rnn_workspace_bytes(dims),), 0xA5, dtype=torch.uint8, device="cuda")
        rnn.rnn_workspace_init(dims, ws)
        rnn.rnn_forward(dims, p, x, None, h, None, ws)
        rnn.rnn_loss(dims, p, h, y, loss, ws)
        rnn.rnn_bptt(dims, p, x, y, h, None, grads, None, ws)
        torch.cuda.synchronize()
        check(p, live, y, h[1:].reshape(T * B, H), loss, grads)


@pytest.mark.parametrize("masked", [[(512, 640)], [(0, 128)], [(130, 500)], [(384, 640), (0, 3)]])
def test_one_window_and_a_stream(masked):
    H, O, T = 40, 640, 12
    p, live, x, y = problem(H, O, T, 1, masked, 5)
    dims = rnn.Dims(O, H, O, T, 1, rnn.INPUT_TOKENS, rnn.ACT_TANH, rnn.LOSS_SOFTMAX_CE, 0)
    h, loss, grads = buffers(p, T, 1, H)
    ws = torch.full((rnn.rnn_window_workspace_bytes(dims),), 0xA5, dtype=torch.uint8, device="cuda")
    rnn.rnn_window_workspace_init(dims, ws)
    rnn.rnn_window(dims, p, x, y, None, None, h, None, loss, grads, None, ws)
    torch.cuda.synchronize()
    check(p, live, y, h[1:].reshape(T, H), loss, grads)
    # one window of the stream: the same loss, and the step against the same gradients
    q = {k: v.clone() for k, v in p.items()}
    losses = torch.full((1,), float("nan"), device="cuda")
    sws = torch.empty(rnn.rnn_train_stream_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    ids = torch.cat([x, y[-1:]]).contiguous()
    rnn.rnn_train_stream(dims, q, ids, 1, 0.5, None, None, losses, sws)
    torch.cuda.synchronize()
    assert rnn.rnn_train_stream_status(sws) == 0
    # (the window's targets are drawn one further on in the same ids, so the two see the same pairs)
    assert abs(float(losses[0]) - float(loss)) <= 1e-4 * abs(float(loss))
    assert torch.isinf(q["c"][~live]).all() and torch.equal(q["V"][:, ~live], p["V"][:, ~live])
    for k in p:
        keep = live if k == "c" else slice(None)
        step = (p[k][keep] - q[k][keep]).double() / 0.5
        ref = grads["d" + k][keep].double()
        assert float((step - ref).abs().max()) <= 1e-3 * float(ref.abs().max()) + 1e-6, k
