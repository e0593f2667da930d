"""Workloads of the recurrent-network training path, as a program that uses the library calls it.

Every case goes through the public entry points of `paper_1211_5590_amd` on device-resident inputs.
Kinds of call:
  window    one truncated-BPTT window of a batch-1 stream in one call (rnn_window)
  stream    many consecutive windows with an SGD update after each in one call (rnn_train_stream)
  calls     rnn_forward -> rnn_loss -> rnn_bptt, the general training pass
  evaluate  rnn_forward -> rnn_loss, the loss of held-out data
  gn        rnn_forward -> rnn_gauss_newton_vec, one curvature product of a Hessian-free optimiser
  mlp       rnn_mlp_train, consecutive SGD batches of the feed-forward classifier
"""
import math

import torch

import paper_1211_5590_amd as rnn

PARAMS = ("Wx", "Wh", "b", "V", "c")
STREAM_LR = 0.1
MLP_LR = 0.005


def _lm(kind, in_dim, hidden, out_dim, seq_len, batch, act="sigmoid", **more):
    return dict(kind=kind, in_dim=in_dim, hidden=hidden, out_dim=out_dim, seq_len=seq_len, batch=batch,
                tokens=True, act=act, loss="ce", bf16x3=False, windows=1, **more)


def listed():
    mlp = dict(kind="mlp", in_dim=784, out_dim=10, act="tanh")
    return [
        # one window of the paper's benchmark shape: what a program that owns its own update rule calls
        # a hundred thousand times; latency of one launch
        dict(_lm("window", 10000, 100, 10000, 10, 1), name="window_10k_h100_t10"),
        # the smallest training pass through the three calls (tests and tutorials): launches only
        dict(_lm("calls", 64, 16, 64, 32, 1), name="calls_tiny_v64_h16_t32"),
        # the paper's benchmark with the update inside: 200 windows of a longer stream per call
        dict(_lm("stream", 10000, 100, 10000, 10, 1), windows=200, name="stream_10k_h100_200_windows"),
        # one long sequence through a larger hidden layer: batch-1 loops over several workgroups
        dict(_lm("calls", 10000, 500, 10000, 100, 1), name="calls_10k_h500_t100"),
        # an ordinary minibatch of a small model: every matrix of the path is of medium size
        dict(_lm("calls", 10000, 200, 10000, 35, 20), name="calls_10k_h200_t35_b20"),
        # the largest language-model step: dense products of 16384 rows
        dict(_lm("calls", 10000, 1024, 10000, 256, 64), name="calls_10k_h1024_t256_b64"),
        # odd and ragged: sizes that are multiples of nothing, on the opt-in split-bf16 output layer
        dict(_lm("calls", 9973, 650, 9973, 70, 33, act="tanh"), bf16x3=True, name="calls_9973_h650_t70_b33_bf16x3"),
        # dense inputs, tanh, mean squared error, very long sequences
        dict(_lm("calls", 128, 256, 128, 4096, 128, act="tanh"), tokens=False, loss="mse",
             name="calls_dense128_h256_t4096_b128"),
        # held-out loss and states of a ragged minibatch, float32 throughout: no backward pass
        dict(_lm("evaluate", 10007, 513, 10007, 100, 19), name="evaluate_10007_h513_t100_b19"),
        # a curvature product on a medium minibatch
        dict(_lm("gn", 10000, 500, 10000, 50, 16), name="gauss_newton_10k_h500_t50_b16"),
        # the feed-forward classifier benchmark: 20 minibatches of 60 through three hidden layers, and
        # 50 single examples through one
        dict(mlp, hidden=1000, n_hidden=3, batch=60, n_batches=20, name="mlp_3x1000_b60"),
        dict(mlp, hidden=500, n_hidden=1, batch=1, n_batches=50, name="mlp_1x500_b1"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["window", "stream", "calls_1", "calls_b", "calls_b", "calls_b", "dense", "evaluate", "gn", "mlp"])
    act = rng.choice(["sigmoid", "tanh"])
    if kind in ("window", "stream"):
        nv = _log(rng, 64, 20000)
        case = _lm(kind, nv, rng.randint(16, 128), nv, rng.randint(4, 32), 1, act=act)
        if kind == "stream":
            case["windows"] = _log(rng, 20, 200)
        return case
    if kind == "mlp":
        return dict(kind="mlp", in_dim=784, out_dim=10, act=act, hidden=_log(rng, 100, 1000), n_hidden=rng.randint(0, 3),
                    batch=_log(rng, 1, 60), n_batches=rng.randint(10, 50))
    if kind == "dense":
        d = _log(rng, 16, 128)
        return dict(_lm("calls", d, _log(rng, 32, 256), d, _log(rng, 64, 4096), _log(rng, 5, 128), act=act),
                    tokens=False, loss=rng.choice(["mse", "mse", "ce"]))
    if kind == "calls_1":
        nv = _log(rng, 64, 10000)
        return _lm("calls", nv, _log(rng, 16, 600), nv, _log(rng, 10, 100), 1, act=act)
    nv = _log(rng, 1000, 10000)
    if kind == "gn":
        return _lm("gn", nv, _log(rng, 64, 600), nv, _log(rng, 10, 60), _log(rng, 1, 24), act=act)
    case = _lm("evaluate" if kind == "evaluate" else "calls", nv, _log(rng, 100, 1024), nv, _log(rng, 10, 256),
               _log(rng, 5, 64), act=act)
    case["bf16x3"] = kind == "calls_b" and rng.random() < 0.3
    return case


# ---- inputs: everything a program holds before the call, drawn from the seed on the device ----------


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    normal = lambda *shape, s=1.0: torch.randn(*shape, generator=g, device="cuda").mul_(s)   # noqa: E731
    if case["kind"] == "mlp":
        rows = case["batch"] * case["n_batches"]
        widths = [case["in_dim"]] + [case["hidden"]] * case["n_hidden"] + [case["out_dim"]]
        return dict(X=torch.rand(rows, case["in_dim"], generator=g, device="cuda"),       # pixel-like inputs
                    y=torch.randint(0, case["out_dim"], (rows,), generator=g, device="cuda", dtype=torch.int32),
                    W=[normal(o, i, s=i ** -0.5) for i, o in zip(widths, widths[1:])],
                    bias=[torch.zeros(o, device="cuda") for o in widths[1:]])
    I, H, O, T, B = (case[k] for k in ("in_dim", "hidden", "out_dim", "seq_len", "batch"))
    p = dict(Wh=normal(H, H, s=H ** -0.5), V=normal(H, O, s=H ** -0.5), b=normal(H, s=0.1), c=normal(O, s=0.1),
             Wx=normal(I, H, s=0.1) if case["tokens"] else normal(H, I, s=I ** -0.5))
    h0 = torch.rand(B, H, generator=g, device="cuda")           # the state carried in from earlier text
    h0 = h0 * 0.9 + 0.05 if case["act"] == "sigmoid" else h0 * 1.8 - 0.9
    d = dict(p=p, h0=h0)
    if case["tokens"]:                                          # Zipf-distributed ids, next-token targets
        cdf = torch.cumsum(torch.arange(1, I + 1, device="cuda", dtype=torch.float64) ** -1.1, 0)
        u = torch.rand(T * case["windows"] + 1, B, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
        d["ids"] = torch.searchsorted(cdf, u).clamp_(max=I - 1).to(torch.int32)
        d["x"], d["y"] = d["ids"][:-1], d["ids"][1:]
    else:
        d["x"] = normal(T, B, I)
        if case["loss"] == "mse":                               # the previous input is to be reproduced
            d["y"] = torch.zeros(T, B, O, device="cuda")
            d["y"][1:] = d["x"][:-1]
        else:
            d["y"] = torch.randint(0, O, (T, B), generator=g, device="cuda", dtype=torch.int32)
    if case["kind"] == "gn":
        d["gamma"] = {k: normal(*v.shape) for k, v in p.items()}
    return d


def _dims(case):
    if case["kind"] == "mlp":
        return rnn.MlpDims(case["in_dim"], case["hidden"], case["n_hidden"], case["out_dim"], case["batch"],
                           rnn.ACT_TANH if case["act"] == "tanh" else rnn.ACT_SIGMOID, 0)
    return rnn.Dims(case["in_dim"], case["hidden"], case["out_dim"], case["seq_len"], case["batch"],
                    rnn.INPUT_TOKENS if case["tokens"] else rnn.INPUT_DENSE,
                    rnn.ACT_TANH if case["act"] == "tanh" else rnn.ACT_SIGMOID,
                    rnn.LOSS_LINEAR_MSE if case["loss"] == "mse" else rnn.LOSS_SOFTMAX_CE,
                    rnn.FLAG_BF16X3_OUTPUT if case["bf16x3"] else 0)


def _bytes_on_gpu(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"], s["dims"] = case["kind"], _dims(case)
    dims = s["dims"]
    if case["kind"] == "mlp":
        s["n"] = case["n_batches"]
        s["losses"] = torch.zeros(s["n"], device="cuda")
        s["ws"] = _bytes_on_gpu(rnn.rnn_mlp_workspace_bytes(dims))
        s["ptrs"] = rnn.mlp_params(s["W"], s["bias"])
        return s
    B, H, T = case["batch"], case["hidden"], case["seq_len"]
    s["h_last"] = torch.zeros(B, H, device="cuda")
    if case["kind"] == "stream":
        s["windows"] = case["windows"]
        s["ids"] = s["ids"].contiguous().view(-1)
        s["losses"] = torch.zeros(case["windows"], device="cuda")
        s["ws"] = _bytes_on_gpu(rnn.rnn_train_stream_workspace_bytes(dims))
        return s
    s["loss"] = torch.zeros(1, device="cuda")
    s["h_all"] = torch.zeros(T + 1, B, H, device="cuda")
    s["grads"] = {"d" + k: torch.zeros_like(v) for k, v in s["p"].items()}
    if case["kind"] == "window":
        s["ws"] = _bytes_on_gpu(rnn.rnn_window_workspace_bytes(dims))
        rnn.rnn_window_workspace_init(dims, s["ws"])
    else:
        size = rnn.rnn_gauss_newton_workspace_bytes if case["kind"] == "gn" else rnn.rnn_workspace_bytes
        s["ws"] = _bytes_on_gpu(size(dims))
        rnn.rnn_workspace_init(dims, s["ws"])
    return s


def run(s):
    kind, dims, ws = s["kind"], s["dims"], s["ws"]
    if kind == "mlp":
        rnn.rnn_mlp_train(dims, s["ptrs"], None, s["X"], s["y"], s["n"], MLP_LR, s["losses"], ws)
        return dict(losses=s["losses"], W=s["W"], b=s["bias"])
    if kind == "stream":
        rnn.rnn_train_stream(dims, s["p"], s["ids"], s["windows"], STREAM_LR, s["h0"], s["h_last"], s["losses"], ws)
        return dict(losses=s["losses"], h_last=s["h_last"], p=s["p"])
    if kind == "window":
        rnn.rnn_window(dims, s["p"], s["x"], s["y"], s["h0"], None, None, s["h_last"], s["loss"], s["grads"], None, ws)
        return dict(loss=s["loss"], h_last=s["h_last"], grads=s["grads"])
    rnn.rnn_forward(dims, s["p"], s["x"], s["h0"], s["h_all"], s["h_last"], ws)
    if kind == "gn":
        rnn.rnn_gauss_newton_vec(dims, s["p"], s["gamma"], s["x"], s["h_all"], rnn.GN_METRIC_LOSS, s["grads"], None, ws)
        return dict(h_all=s["h_all"], Gv=s["grads"])
    rnn.rnn_loss(dims, s["p"], s["h_all"], s["y"], s["loss"], ws)
    if kind == "evaluate":
        return dict(loss=s["loss"], h_all=s["h_all"])
    rnn.rnn_bptt(dims, s["p"], s["x"], s["y"], s["h_all"], None, s["grads"], None, ws)
    return dict(loss=s["loss"], h_all=s["h_all"], grads=s["grads"])


def work(case):
    f = 4.0
    if case["kind"] == "mlp":
        widths = [case["in_dim"]] + [case["hidden"]] * case["n_hidden"] + [case["out_dim"]]
        sizes = [a * b for a, b in zip(widths, widths[1:])]
        rows = case["batch"] * case["n_batches"]
        # forward and dW for every layer, dX for all but the first; the model read and written once
        flops = rows * (4.0 * sum(sizes) + 2.0 * sum(sizes[1:]))
        return dict(bytes=f * (rows * (case["in_dim"] + 1) + 2 * (sum(sizes) + sum(widths[1:])) + case["n_batches"]), flops=flops)
    I, H, O = case["in_dim"], case["hidden"], case["out_dim"]
    N, B = case["seq_len"] * case["batch"] * case["windows"], case["batch"]
    core, out = H * H + H + H * O + O, (O if case["loss"] == "mse" else 1) * N
    x = N * (H + 1) if case["tokens"] else N * I + I * H        # gathered rows and their ids, or all inputs and Wx
    if case["kind"] == "stream":
        rows = min(N, I) * H
        return dict(bytes=f * (N + 2 * core + 2 * rows + case["windows"] + 2 * H), flops=6.0 * N * H * O + 6.0 * N * H * H)
    flops, moved = 2.0 * N * H * H + 2.0 * N * H * O, core + x + out + B * H
    if not case["tokens"]:
        flops += 2.0 * N * H * I
    if case["kind"] == "evaluate":
        return dict(bytes=f * (moved + N * H), flops=flops)
    grads = core + I * H
    states = B * H if case["kind"] == "window" else N * H
    flops += 4.0 * N * H * H + 4.0 * N * H * O + (0.0 if case["tokens"] else 2.0 * N * H * I)
    if case["kind"] == "gn":   # a second forward sweep and the direction's own products
        flops += 4.0 * N * H * H + 4.0 * N * H * O
        moved += core + N * H - out
    return dict(bytes=f * (moved + grads + states), flops=flops)


def tolerance(case):
    # about four times the distance from the 64-bit result over the ranges above; the largest is that of
    # dV of the largest step (1e-5: sums over 16384 rows that nearly cancel)
    if case["kind"] in ("window", "stream", "mlp"):
        return dict(rel=1e-5, max=1e-4)
    return dict(rel=4e-5, max=2e-3 if case["bf16x3"] else 4e-4)


# ---- the same outputs in 64 bits, plain torch ------------------------------------------------------


def _act(a, kind):
    return torch.sigmoid(a) if kind == "sigmoid" else torch.tanh(a)


def _slope(h, kind):
    return h * (1 - h) if kind == "sigmoid" else 1 - h * h


def _forward(p, x, h0, act, tokens):
    U = (p["Wx"][x.long()] if tokens else x @ p["Wx"].t()) + p["b"]
    h_all = torch.empty((x.shape[0] + 1,) + h0.shape, dtype=torch.float64, device=h0.device)
    h_all[0] = h0
    WhT = p["Wh"].t().contiguous()
    for t in range(x.shape[0]):
        h_all[t + 1] = _act(U[t] + h_all[t] @ WhT, act)
    return h_all


def _loss_and_dz(p, h_all, y, loss):
    H = h_all.shape[2]
    Z = h_all[1:].reshape(-1, H) @ p["V"] + p["c"]
    N = Z.shape[0]
    if loss == "mse":
        d = Z - y.reshape(Z.shape)
        return d.square().mean(), d.mul_(2.0 / d.numel()), None
    target = y.reshape(-1).long()
    lse = torch.logsumexp(Z, 1)
    value = (lse - Z.gather(1, target[:, None])[:, 0]).mean()
    P = Z.sub_(lse[:, None]).exp_()
    dZ = P / N
    dZ[torch.arange(N, device=dZ.device), target] -= 1.0 / N
    return value, dZ, P


def _backward(p, x, h_all, dZ, act, tokens):
    T, B, H = x.shape[0], h_all.shape[1], h_all.shape[2]
    Hs = h_all[1:].reshape(-1, H)
    G = (dZ @ p["V"].t()).reshape(T, B, H)
    D = torch.empty_like(G)
    nxt = torch.zeros_like(h_all[0])
    for t in range(T - 1, -1, -1):
        D[t] = (G[t] + nxt) * _slope(h_all[t + 1], act)
        nxt = D[t] @ p["Wh"]
    Df = D.reshape(-1, H)
    if tokens:
        dWx = torch.zeros_like(p["Wx"]).index_add_(0, x.reshape(-1).long(), Df)
    else:
        dWx = Df.t() @ x.reshape(T * B, -1)
    return dict(dWx=dWx, dWh=Df.t() @ h_all[:-1].reshape(-1, H), db=Df.sum(0), dV=Hs.t() @ dZ, dc=dZ.sum(0))


def _exact_mlp(case, d):
    W, b = [w.double() for w in d["W"]], [v.double() for v in d["bias"]]
    n, losses = case["batch"], []
    for k in range(case["n_batches"]):
        a = [d["X"][k * n:(k + 1) * n].double()]
        for w, v in zip(W[:-1], b[:-1]):
            a.append(_act(a[-1] @ w.t() + v, case["act"]))
        z, t = a[-1] @ W[-1].t() + b[-1], d["y"][k * n:(k + 1) * n].long()
        lse = torch.logsumexp(z, 1)
        losses.append((lse - z.gather(1, t[:, None])[:, 0]).mean())
        dz = torch.exp(z - lse[:, None])
        dz[torch.arange(n, device=dz.device), t] -= 1.0
        dz = dz / n
        for l in range(len(W) - 1, -1, -1):
            below = (dz @ W[l]) * _slope(a[l], case["act"]) if l else None
            W[l], b[l] = W[l] - MLP_LR * (dz.t() @ a[l]), b[l] - MLP_LR * dz.sum(0)
            dz = below
    return dict(losses=torch.stack(losses), W=W, b=b)


def exact(case, seed):
    d = _inputs(case, seed)
    if case["kind"] == "mlp":
        return _exact_mlp(case, d)
    wide = lambda v: v.double() if v.is_floating_point() else v   # noqa: E731
    p, act, tokens = {k: v.double() for k, v in d["p"].items()}, case["act"], case["tokens"]
    h, T = d["h0"].double(), case["seq_len"]
    if case["kind"] == "stream":
        losses = []
        for w in range(case["windows"]):
            x, y = d["x"][w * T:(w + 1) * T], d["y"][w * T:(w + 1) * T]
            h_all = _forward(p, x, h, act, tokens)
            value, dZ, _ = _loss_and_dz(p, h_all, y, case["loss"])
            g = _backward(p, x, h_all, dZ, act, tokens)
            p = {k: p[k] - STREAM_LR * g["d" + k] for k in PARAMS}
            h = h_all[-1]
            losses.append(value)
        return dict(losses=torch.stack(losses), h_last=h, p=p)
    x, y = wide(d["x"]), wide(d["y"])
    h_all = _forward(p, x, h, act, tokens)
    if case["kind"] == "gn":
        return dict(h_all=h_all, Gv=_exact_gn(p, {k: v.double() for k, v in d["gamma"].items()}, x, y, h_all, act))
    value, dZ, _ = _loss_and_dz(p, h_all, y, case["loss"])
    if case["kind"] == "evaluate":
        return dict(loss=value.reshape(1), h_all=h_all)
    grads = _backward(p, x, h_all, dZ, act, tokens)
    if case["kind"] == "window":
        return dict(loss=value.reshape(1), h_last=h_all[-1], grads=grads)
    return dict(loss=value.reshape(1), h_all=h_all, grads=grads)


def _exact_gn(p, gamma, x, y, h_all, act):
    T, H = x.shape[0], h_all.shape[2]
    Hs = h_all[1:].reshape(-1, H)
    C = gamma["Wx"][x.long()] + gamma["b"] + h_all[:-1] @ gamma["Wh"].t()
    R = torch.empty_like(h_all[1:])
    prev = torch.zeros_like(h_all[0])
    for t in range(T):
        prev = R[t] = _slope(h_all[t + 1], act) * (C[t] + prev @ p["Wh"].t())
    Rz = R.reshape(-1, H) @ p["V"] + Hs @ gamma["V"] + gamma["c"]
    _, _, P = _loss_and_dz(p, h_all, y, "ce")
    u = P * (Rz - (P * Rz).sum(1, keepdim=True)) / Rz.shape[0]
    return _backward(p, x, h_all, u, act, True)
