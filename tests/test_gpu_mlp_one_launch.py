"""The one-launch form of the classifier training (at most one hidden layer, 64 rows, 16 classes) at the
edges of its tiles and of the sizes it serves, on both sides of each, against the float64 oracle."""
import numpy as np
import pytest
import torch

import paper_1211_5590_amd as rnn
import rnn_inputs as ri
from oracle import mlp
from test_gpu_mlp import check, run_gpu

pytestmark = pytest.mark.gpu

# in_dim, hidden (0: none), classes, batch
SIZES = [(4, 0, 1, 1), (16, 0, 16, 2), (256, 0, 10, 16), (260, 0, 10, 17), (896, 0, 10, 64), (900, 0, 10, 64),
         (8, 1, 2, 1), (20, 16, 3, 2), (128, 17, 16, 33), (784, 33, 10, 1), (784, 100, 10, 32), (132, 500, 10, 64),
         (784, 0, 10, 21), (784, 126, 10, 21), (64, 1024, 16, 64), (64, 1025, 10, 3), (252, 40, 16, 65), (784, 1000, 10, 1), (784, 300, 7, 9)]


@pytest.mark.parametrize("I,H,O,B", SIZES)
def test_edges_of_the_one_launch_form(I, H, O, B):
    for act in (ri.ACT_TANH, ri.ACT_SIGMOID):
        case = ri.make_mlp_case(I, H, 1 if H else 0, O, B, n_batches=5, act=act, bias_std=0.2, seed=I + H + B)
        # a step that does not overshoot: |x|^2 is about I / 3.  (A loss is logsumexp(z) - z[y], two float32
        # numbers of the size of z: where training diverges to losses near 0 at |z| of 10, their
        # difference keeps 10 2^-24 / loss of its digits, beyond any relative tolerance.)
        lr = min(0.05, 4.0 / I)
        check(run_gpu(case, lr), mlp.train(case, lr), case)


@pytest.mark.parametrize("hidden", [0, 40])
def test_more_batches_than_one_launch_takes(hidden):
    case = ri.make_mlp_case(12, hidden, 1 if hidden else 0, 4, 3, n_batches=1030, bias_std=0.1, seed=5)
    got, ref = run_gpu(case, 0.02), mlp.train(case, 0.02)
    np.testing.assert_allclose(got["losses"], ref["losses"], rtol=2e-4)
    for l in range(len(case["W"])):
        np.testing.assert_allclose(got["W"][l], ref["W"][l], rtol=0, atol=2e-4 * np.abs(ref["W"][l]).max())


def test_two_streams_and_a_captured_call_repeat_exactly():
    case = ri.make_mlp_case(100, 60, 1, 10, 8, n_batches=6, bias_std=0.1, seed=9)
    first = run_gpu(case, 0.1)
    dims = rnn.MlpDims.of(case)
    sets = []
    for _ in range(2):
        d = lambda a: torch.from_numpy(a.copy()).cuda()   # noqa: E731
        sets.append(dict(W=[d(w) for w in case["W"]], b=[d(v) for v in case["b"]], X=d(case["X"]), y=d(case["y"]),
                         losses=torch.zeros(6, device="cuda"),
                         ws=torch.empty(rnn.rnn_mlp_workspace_bytes(dims), dtype=torch.uint8, device="cuda"),
                         stream=torch.cuda.Stream()))
    torch.cuda.synchronize()
    for s in sets:
        rnn.rnn_mlp_train(dims, s["W"], s["b"], s["X"], s["y"], 6, 0.1, s["losses"], s["ws"], stream=s["stream"])
    torch.cuda.synchronize()
    for s in sets:
        assert np.array_equal(s["losses"].cpu().numpy(), first["losses"])
        for l in range(2):
            assert np.array_equal(s["W"][l].cpu().numpy(), first["W"][l])
    s = sets[0]
    W0, b0 = [torch.from_numpy(w.copy()).cuda() for w in case["W"]], [torch.from_numpy(v.copy()).cuda() for v in case["b"]]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rnn.rnn_mlp_train(dims, s["W"], s["b"], s["X"], s["y"], 6, 0.1, s["losses"], s["ws"])
    for _ in range(3):
        for w, w0 in zip(s["W"], W0):
            w.copy_(w0)
        for v, v0 in zip(s["b"], b0):
            v.copy_(v0)
        s["losses"].fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(s["losses"].cpu().numpy(), first["losses"])
        assert np.array_equal(s["W"][0].cpu().numpy(), first["W"][0])


@pytest.mark.parametrize("I,H,L,O,B", ((1, 2, 2, 3, 1), (3, 5, 3, 2, 16), (63, 65, 2, 17, 17), (66, 255, 2, 10, 32), (257, 61, 3, 16, 33),
                                       (64, 258, 2, 5, 64), (130, 67, 2, 10, 65)))
def test_the_update_of_deep_classifiers_at_ragged_rows(I, H, L, O, B):
    """Rows of the weights that end inside a lane's 16-byte piece, in every form the batch size picks."""
    case = ri.make_mlp_case(I, H, L, O, B, n_batches=4, act=ri.ACT_TANH, bias_std=0.2, seed=I + H + B)
    lr = min(0.05, 4.0 / I)
    check(run_gpu(case, lr), mlp.train(case, lr), case)


@pytest.mark.parametrize("I,H,B,m", ((784, 30, 10, 4), (20, 9, 3, 1), (784, 40, 33, 32), (260, 16, 60, 17), (36, 20, 17, 16),
                                     (784, 33, 21, 20), (256, 17, 32, 7)))
def test_an_infinite_input_stays_in_its_own_example(I, H, B, m):
    """Saturating hidden units keep the logits of an example with an infinite input finite: the batch's loss is finite,
    and the step is not a number in the column of that input alone (0 times infinity), as in the oracle."""
    for k in (0, I - 1):
        case = ri.make_mlp_case(I, H, 1, 10, B, n_batches=1, act=ri.ACT_TANH, bias_std=0.2, seed=I + H + B)
        case["X"][m, k] = np.inf
        with np.errstate(invalid="ignore"):
            ref = mlp.train(case, 0.05)
        got = run_gpu(case, 0.05)
        assert np.isfinite(ref["losses"]).all()
        np.testing.assert_allclose(got["losses"], ref["losses"], rtol=1e-4)
        for l in range(2):
            nan = np.isnan(ref["W"][l])
            assert l == 1 or (nan[:, k].all() and nan.sum() == H)
            assert np.array_equal(np.isnan(got["W"][l]), nan)
            assert np.abs(got["W"][l] - ref["W"][l])[~nan].max() <= 1e-4 * np.abs(ref["W"][l][~nan]).max()
