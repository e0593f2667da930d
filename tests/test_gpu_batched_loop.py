"""The batched loop with register-resident weights at every number of 32-unit slabs it is built for, on
both sides of every slab edge, with missing batch rows, both directions and activations, against the
oracle; and infinities, which its three-way bf16 split cannot hold."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_5590_amd as rnn
import rnn_inputs as ri
from gpu_harness import Runner, compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [1, 2, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 255, 256])
def test_every_slab_count(H):
    for n, (B, T) in enumerate(((5, 1), (8, 2), (7, 12))):
        case = ri.make_case(40, H, 30, T, B, act=n % 2, with_h0=n != 1, with_dh_last=n >= 1,
                            wdist=("normal", 0.7 / np.sqrt(H)), bias_std=0.1, seed=700 + 5 * H + n)
        r = Runner(case)
        assert rnn.rnn_recurrence_variant(r.dims) == "batch_mfma"
        r.step()
        compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


@pytest.mark.parametrize("where", ["matrix", "state", "large"])
def test_infinities_give_what_float32_gives(where):
    H, B, T = 70, 6, 3
    g = torch.Generator().manual_seed(1)
    Wh = torch.rand(H, H, generator=g) * 0.2 - 0.1
    h = torch.rand(B, H, generator=g) * 0.5 + 0.2
    U = torch.rand(T, B, H, generator=g) - 0.5
    if where == "matrix":
        Wh[3, 5], Wh[9, 60] = float("inf"), float("-inf")
    elif where == "state":
        h[2, 7] = float("inf")
        Wh[:, 7] = Wh[:, 7].abs() + 0.01
    else:
        Wh[4, 4] = 3.4e38                      # rounds to infinity in bf16
    p = dict(Wx=torch.eye(H).cuda(), Wh=Wh.cuda(), b=torch.zeros(H).cuda(), V=torch.zeros(H, 2).cuda(), c=torch.zeros(2).cuda())
    dims = rnn.Dims(H, H, 2, T, B, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    hist = torch.zeros(T + 1, B, H, device="cuda")
    rnn.rnn_forward(dims, p, U.cuda(), h.cuda(), hist, None, ws)
    got = hist.cpu()
    for t in range(T):
        ref = torch.tanh(got[t] @ Wh.t() + U[t])
        assert torch.equal(torch.isnan(got[t + 1]), torch.isnan(ref)), t
        fine = ~torch.isnan(ref)
        assert float((got[t + 1][fine] - ref[fine]).abs().max()) < 1e-5


@pytest.mark.parametrize("H", [30, 70, 250])
def test_a_state_beyond_bf16s_range_against_weights_of_zero(H):
    """3.4e38 is a float32 that rounds to infinity in bf16: times a weight of zero it adds nothing."""
    B, T = 6, 5
    big = 3.4e38
    g = torch.Generator().manual_seed(2)
    Wh = torch.rand(H, H, generator=g) * 0.2 - 0.1
    Wh[:, 7] = 0.0
    Wh[5, 7] = 1e-38                             # and one that leaves something of it
    U = torch.rand(T, B, H, generator=g) - 0.5
    p = dict(Wx=torch.eye(H).cuda(), Wh=Wh.cuda(), b=torch.zeros(H).cuda(), V=torch.zeros(H, 2).cuda(), c=torch.zeros(2).cuda())
    dims = rnn.Dims(H, H, 2, T, B, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    h0 = torch.rand(B, H, generator=g) * 0.5
    h0[2, 7], h0[4, 7] = big, -big
    for last_only in (False, True):
        hist = None if last_only else torch.zeros(T + 1, B, H, device="cuda")
        last = torch.zeros(B, H, device="cuda")
        rnn.rnn_forward(dims, p, U.cuda(), h0.cuda(), hist, last, ws)
        h = h0.double()
        for t in range(T):
            h = torch.tanh(h @ Wh.double().t() + U[t].double())
            if not last_only:
                assert float((hist[t + 1].cpu().double() - h).abs().max()) < 2e-5, t
        assert float((last.cpu().double() - h).abs().max()) < 2e-5
    # reverse loop: states of zero (slope 1), the incoming gradient is the large number
    Wh[7, :] = 0.0
    Wh[7, 5] = 1e-38
    p["Wh"] = Wh.cuda()
    hist = torch.zeros(T + 1, B, H, device="cuda")
    dh = torch.rand(B, H, generator=g)
    dh[1, 7] = big
    loss = torch.zeros(1, device="cuda")
    grads = {"d" + k: torch.zeros_like(v) for k, v in p.items()}
    dh0 = torch.zeros(B, H, device="cuda")
    Y = torch.zeros(T, B, 2, device="cuda")
    rnn.rnn_loss(dims, p, hist, Y, loss, ws)
    rnn.rnn_bptt(dims, p, torch.zeros(T, B, H, device="cuda"), Y, hist, dh.cuda(), grads, dh0, ws)
    d = dh.double()
    for t in range(T):
        d = d @ Wh.double()
    assert float((dh0.cpu().double() - d).abs().max()) <= 1e-5 * float(d.abs().max())


@pytest.mark.parametrize("H", [70, 256])
def test_an_infinity_of_one_state_costs_that_step_only(H):
    """The steps that take float32 products from memory are those whose state holds the infinity: one, as tanh is finite.
    (512 steps of the ordinary form are 15 of such a step, so a factor of 3 is far from both outcomes.)"""
    B, T = 8, 512
    g = torch.Generator(device="cuda").manual_seed(4)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") - 0.5   # noqa: E731
    p = dict(Wx=rand(H, 8), Wh=rand(H, H) * 0.2, b=rand(H), V=rand(H, 2), c=rand(2))
    dims = rnn.Dims(8, H, 2, T, B, rnn.INPUT_DENSE, rnn.ACT_TANH, rnn.LOSS_LINEAR_MSE, 0)
    ws = torch.empty(rnn.rnn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    rnn.rnn_workspace_init(dims, ws)
    X, h0, hist = rand(T, B, 8), rand(B, H), torch.zeros(T + 1, B, H, device="cuda")
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best():
        times = []
        for _ in range(6):
            t0.record()
            rnn.rnn_forward(dims, p, X, h0, hist, None, ws)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)
    finite = best()
    h0[1, 3] = float("inf")
    assert best() < 3.0 * finite
