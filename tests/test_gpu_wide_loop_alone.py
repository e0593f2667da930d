"""The wide loop when not all workgroups of a group come: one of them closes the group's roll and runs its recurrence by itself.
And when all come but a wait for a state expires: the launch ends, with status 1."""
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_1211_5590_amd as rnn
import rnn_inputs as ri
from gpu_harness import Runner, compare

pytestmark = pytest.mark.gpu


def make(H, B, T, kind, seed=0):
    return ri.make_case(in_dim=92, hidden=H, out_dim=72, seq_len=T, batch=B, act=kind, input_kind=kind, with_h0=kind == 0,
                        with_dh_last=kind == 1, wdist=("normal", 0.5 / np.sqrt(H)), bias_std=0.1, seed=7100 + 11 * H + B + seed)


@pytest.mark.parametrize("H,B,T", ((257, 5, 10), (301, 1, 16), (512, 33, 11), (515, 64, 12), (1023, 6, 10), (1024, 61, 10),
                                   (255, 127, 64)))
@pytest.mark.parametrize("kind", (0, 1))
def test_one_workgroup_runs_a_group_whose_others_are_missing(H, B, T, kind):
    case = make(H, B, T, kind)
    r = Runner(case)
    print(f"H={H} B={B} T={T} kind={kind}", flush=True)
    assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
    ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
    groups = (B + 3) // 4
    # the roll is closed as soon as somebody looks at it, and after 300 us
    for wait in (0, 300):
        rnn.rnn_test_roll_call(wait, 1)
        try:
            r.forward()
            assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == groups
            r.loss_()
            r.bptt()
        finally:
            rnn.rnn_test_roll_call()
        assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == groups
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), ref)
    r.step()
    assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == 0
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    compare(r.results(), ref)


@pytest.mark.parametrize("H,B,T", ((260, 7, 40), (500, 30, 43), (513, 5, 40), (256, 128, 70), (600, 40, 41), (1024, 64, 40)))
@pytest.mark.parametrize("kind", (0, 1))
def test_smallest_wait_limit_on_every_width_of_the_wide_loop_never_hangs(H, B, T, kind):
    """16, 32 and 64 columns per workgroup, more and fewer steps than the carrier takes between two looks at the abort word.  With a
    bound of one poll a wait for a state may expire (status 1, results invalid) or not (status 0, right results); the first wait,
    for the group, is not bounded by it."""
    case = make(H, B, T, kind, seed=3)
    ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
    r = Runner(case)
    assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
    seen = []
    rnn.rnn_set_wait_limit(1)
    try:
        for _ in range(3):
            rnn.rnn_workspace_init(r.dims, r.ws)
            r.step()
            seen.append(rnn.rnn_workspace_status(r.dims, r.ws))
            assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == 0
            if seen[-1] == 0:
                compare(r.results(), ref)
    finally:
        rnn.rnn_set_wait_limit(0)
    print(f"H={H} B={B} T={T} kind={kind}: status {seen}", flush=True)
    assert set(seen) <= {0, 1}
    rnn.rnn_workspace_init(r.dims, r.ws)
    r.step()
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    compare(r.results(), ref)
    if 1 not in seen:
        pytest.skip("no wait expired, so nothing was seen of what follows")


@pytest.mark.parametrize("H,B,T", ((500, 32, 40), (1024, 64, 12)))
def test_workgroups_that_come_late_to_a_closed_roll(H, B, T):
    """A loop of 16 workgroups on another stream holds two compute units of every die, and the first workgroup that looks closes its
    group's roll: those that start later find it closed and leave.  Right results, whichever groups that was."""
    case = make(H, B, T, 0, seed=5)
    ref = oracle.fwd_bptt(case, h0=case.get("h0"))
    r = Runner(case)
    long = Runner(make(192, 64, 4000, 1))
    assert rnn.rnn_recurrence_variant(long.dims) == "batch_mfma"
    r.step()
    other = torch.cuda.Stream()
    alone = 0
    rnn.rnn_test_roll_call(0)
    try:
        for _ in range(5):
            with torch.cuda.stream(other):
                long.forward()
            r.forward()
            n = rnn.rnn_workspace_groups_alone(r.dims, r.ws)
            r.loss_()
            r.bptt()
            print("groups alone:", n, rnn.rnn_workspace_groups_alone(r.dims, r.ws), flush=True)
            alone += n
            assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
            compare(r.results(), ref)
            torch.cuda.synchronize()
    finally:
        rnn.rnn_test_roll_call()
    if alone == 0:
        pytest.skip("every group came together")


@pytest.mark.parametrize("H,B,T", ((193, 3, 64), (256, 30, 64), (255, 127, 64), (257, 5, 17), (384, 32, 10), (384, 33, 10), (512, 33, 11),
                                   (515, 64, 12), (640, 17, 10), (769, 40, 10), (897, 64, 10), (1023, 6, 10), (1024, 61, 10)))
@pytest.mark.parametrize("kind", (0, 1))
def test_a_group_run_alone_gives_the_same_bits(H, B, T, kind):
    """Which way a group is computed depends on what else the GPU does, the results do not: every number of K per wavefront and of
    columns per workgroup, tokens and dense input, with and without an initial state and a gradient from later."""
    r = Runner(make(H, B, T, kind, seed=9))
    assert rnn.rnn_recurrence_variant(r.dims) == "xcd_mfma"
    r.step()
    assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == 0
    together = r.results()
    rnn.rnn_test_roll_call(0, 1)
    try:
        r.step()
    finally:
        rnn.rnn_test_roll_call()
    assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == (B + 3) // 4
    alone = r.results()
    for name, v in together.items():
        assert np.array_equal(v, alone[name]), name


@pytest.mark.parametrize("beside", ("wide_loop", "train_stream", "grid_loop", "classifier"))
def test_launches_that_wait_inside_take_turns(beside):
    """A wide loop on one stream beside, on another, each launch of the library whose workgroups wait for each other: they share the
    chip one after the other, so no group is ever run alone and no wait expires."""
    case = make(1000, 64, 30, 0, seed=2)
    ref = oracle.fwd_bptt(case, h0=case.get("h0"))
    r = Runner(case)
    status = lambda: 0                                       # noqa: E731
    if beside == "wide_loop":
        other = Runner(make(500, 32, 2500, 1))
        call, status = other.forward, lambda: rnn.rnn_workspace_status(other.dims, other.ws)   # noqa: E731
    elif beside == "grid_loop":
        other = Runner(make(900, 1, 1200, 1))
        assert rnn.rnn_recurrence_variant(other.dims) == "grid_resident"
        call, status = other.forward, lambda: rnn.rnn_workspace_status(other.dims, other.ws)   # noqa: E731
    elif beside == "train_stream":
        stream = ri.make_config("C2", windows=400)
        dims = rnn.Dims.of(stream)
        params = {k: torch.from_numpy(stream[k]).cuda() for k in ("Wx", "Wh", "b", "V", "c")}
        ids = torch.from_numpy(np.ascontiguousarray(ri.stream_ids(stream)).reshape(-1)).cuda()
        losses = torch.empty(400, device="cuda")
        ws = torch.zeros(rnn.rnn_train_stream_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
        call = lambda: rnn.rnn_train_stream(dims, params, ids, 400, 0.01, None, None, losses, ws)   # noqa: E731
        status = lambda: rnn.rnn_train_stream_status(ws)    # noqa: E731
    else:
        mlp = dict(in_dim=784, hidden=500, n_hidden=1, out_dim=10, batch=1, act=0)
        dims = rnn.MlpDims.of(mlp)
        W = [torch.randn(500, 784, device="cuda") / 28, torch.randn(10, 500, device="cuda") / 23]
        b = [torch.zeros(500, device="cuda"), torch.zeros(10, device="cuda")]
        X, y = torch.rand(400, 784, device="cuda"), torch.zeros(400, dtype=torch.int32, device="cuda")
        losses = torch.empty(400, device="cuda")
        ws = torch.zeros(rnn.rnn_mlp_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
        call = lambda: rnn.rnn_mlp_train(dims, W, b, X, y, 400, 0.01, losses, ws)   # noqa: E731
    call()
    r.step()
    torch.cuda.synchronize()
    errors, done = [], threading.Event()

    def work():
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                while not done.is_set():
                    call()
                    torch.cuda.current_stream().synchronize()
        except Exception as e:                              # noqa: BLE001 -- shown by the assert below
            errors.append(e)

    t = threading.Thread(target=work)
    t.start()
    alone = []
    try:
        rnn.rnn_test_roll_call(300)      # much longer than the small kernels in between, much shorter than a launch of the other stream
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                r.forward()
                alone.append(rnn.rnn_workspace_groups_alone(r.dims, r.ws))
                r.loss_()
                r.bptt()
                alone.append(rnn.rnn_workspace_groups_alone(r.dims, r.ws))
            torch.cuda.current_stream().synchronize()
    finally:
        rnn.rnn_test_roll_call()
        done.set()
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    assert alone == [0] * 40, alone
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0 and status() == 0
    compare(r.results(), ref)


@pytest.mark.parametrize("replayed", ("wide_loop", "grid_loop"))
def test_eager_wide_loops_beside_a_replayed_graph(replayed):
    """A graph's launches take no turns: they may find the chip partly taken by an eager loop and the other way round.  Both end, with
    right results and status 0, whichever groups were run alone."""
    eager, graph = Runner(make(600, 40, 40, 0, seed=6)), Runner(make(500, 33, 40, 1) if replayed == "wide_loop" else make(900, 1, 40, 1))
    assert rnn.rnn_recurrence_variant(graph.dims) == ("xcd_mfma" if replayed == "wide_loop" else "grid_resident")
    refs = [oracle.fwd_bptt(r.case, h0=r.case.get("h0"), dh_last=r.case.get("dh_last")) for r in (eager, graph)]
    eager.step()
    graph.step()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(captured, stream=side):
        graph.forward(); graph.loss_(); graph.bptt()
    errors, alone = [], []

    def work():
        try:
            with torch.cuda.stream(side):
                for _ in range(20):
                    captured.replay()
                    side.synchronize()
        except Exception as e:                              # noqa: BLE001 -- shown by the assert below
            errors.append(e)

    t = threading.Thread(target=work)
    t.start()
    try:
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                eager.forward()
                alone.append(rnn.rnn_workspace_groups_alone(eager.dims, eager.ws))
                eager.loss_(); eager.bptt()
            torch.cuda.current_stream().synchronize()
    finally:
        t.join()
    torch.cuda.synchronize()
    print("groups alone:", alone, flush=True)
    assert not errors, errors
    for r, ref in zip((eager, graph), refs):
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), ref)


@pytest.mark.parametrize("H,B,T,kind,wide", ((200, 20, 35, 0, False), (193, 1, 64, 1, False), (256, 2, 2047, 0, False),
                                             (256, 2, 2048, 0, True), (193, 5, 2047, 1, False), (193, 5, 2048, 1, True), (256, 127, 70, 0, False),
                                             (257, 5, 16, 0, True)))
def test_which_loop_a_captured_call_takes(H, B, T, kind, wide):
    """A wide loop in a graph is a cooperative launch, so that shorter sequences of up to 256 units stay with the loop of one workgroup
    per 4 rows.  It leaves the wide loop's words in the workspace as the last eager call left them."""
    case = make(H, B, T, kind, seed=4)
    ref = oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last"))
    r = Runner(case)
    r.step()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        r.forward(); r.loss_(); r.bptt()
    for rep in range(3):
        rnn.rnn_test_roll_call(0, 1)                        # an eager call between the replays, all groups alone
        try:
            r.step()
        finally:
            rnn.rnn_test_roll_call()
        assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == (B + 3) // 4
        for t in (r.h_all, r.h_last, r.loss, r.dh0, *r.grads.values()):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert rnn.rnn_workspace_groups_alone(r.dims, r.ws) == (0 if wide else (B + 3) // 4)
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), ref)


def test_wide_loops_of_two_threads_on_two_streams():
    """Each loop needs all compute units of the dies it uses: those of two streams take turns."""
    cases = [make(600, 40, 40, 0), make(1000, 64, 30, 1)]
    refs = [oracle.fwd_bptt(c, h0=c.get("h0"), dh_last=c.get("dh_last")) for c in cases]
    runners = [Runner(c) for c in cases]
    torch.cuda.synchronize()
    errors = []

    def work(r):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(10):
                    r.forward(); r.loss_(); r.bptt()
                torch.cuda.current_stream().synchronize()
        except Exception as e:                              # noqa: BLE001 -- shown by the assert below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(r,)) for r in runners]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for r, ref in zip(runners, refs):
        assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
        compare(r.results(), ref)
