"""The wide loop when not all workgroups of a group come: one of them runs the group's recurrence by itself.  With a wait limit of
one poll the first workgroup of a group waits for nobody."""
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
    rnn.rnn_set_wait_limit(1)
    try:
        r.step()
    finally:
        rnn.rnn_set_wait_limit(0)
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))
    r.step()
    assert rnn.rnn_workspace_status(r.dims, r.ws) == 0
    compare(r.results(), oracle.fwd_bptt(case, h0=case.get("h0"), dh_last=case.get("dh_last")))


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
