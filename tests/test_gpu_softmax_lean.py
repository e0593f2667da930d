"""The probabilities of a softmax over thousands of classes have no error in common: dc of classes that are no target is their mean
over the rows, and its relative error, averaged over the classes, is what the probabilities of all rows share.

Bound: the log-sum-exp of a row (8 to 16 here) is rounded to float32 by at most 2^-21, independently from row to row, so the mean over N
rows is within 5 * 2^-21 / sqrt(3 N) of nothing (5 standard deviations); the exponential's own mean error is below 2^-27.
The loss is a mean that is rounded once: 2^-23 of itself, and the rows' roundings on the mean."""
import numpy as np
import pytest
import torch

import paper_1211_5590_amd as rnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,O", [(700, 64, 10000), (900, 40, 30001), (700, 500, 10000)])   # (the last one's logits: K cut or not by the plan)
def test_probabilities_share_no_error(N, H, O):
    g = torch.Generator(device="cuda").manual_seed(N + O)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    p = dict(Wx=rand(4, H), Wh=rand(H, H) * 0.1, b=rand(H), V=rand(H, O) / H ** 0.5, c=rand(O) * 0.1)
    dims = rnn.Dims(4, H, O, 1, N, rnn.INPUT_TOKENS, rnn.ACT_SIGMOID, rnn.LOSS_SOFTMAX_CE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h = torch.rand(2, N, H, generator=g, device="cuda")
    x = torch.zeros(1, N, dtype=torch.int32, device="cuda")
    y = torch.randint(0, O // 2, (1, N), generator=g, device="cuda", dtype=torch.int32)
    loss = torch.zeros(1, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    rnn.rnn_loss(dims, p, h, y, loss, ws)
    rnn.rnn_bptt(dims, p, x, y, h, None, grads, None, ws)
    Z = h[1].double() @ p["V"].double() + p["c"].double()
    lse = torch.logsumexp(Z, 1)
    dc = torch.exp(Z - lse[:, None]).mean(0)[O // 2:]
    shared = float(((grads["dc"][O // 2:].double() - dc) / dc).mean())
    assert abs(shared) <= 5 * 2.0 ** -21 / np.sqrt(3.0 * N) + 2.0 ** -27, shared
    want = float((lse - Z.gather(1, y[0].long()[:, None])[:, 0]).mean())
    assert abs(float(loss) - want) <= 2.0 ** -23 * want + 5 * 2.0 ** -21 / np.sqrt(3.0 * N)
